"""Meshes of one tile bucket: the sums pass and the sort share out the catalog in runs of
1024 particles, one or four at a time; sizes at the edges of a run, of a workgroup's share
and of four runs, against a painting by torch in FP64 and the same sums."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402
from perf import cases  # noqa: E402


def _catalog(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.randint(0, 1 << 32, (3, n), generator=g, device="cuda", dtype=torch.int64)
    return (p - ((p >> 31) << 32)).to(torch.int32), 0.5 + torch.rand(n, generator=g, device="cuda")


@pytest.mark.parametrize("nran", [1, 1023, 1024, 1025, 2049, 262143, 262144, 262145, 1048576, 1048577, 1311745])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n", [16, 64])
def test_runs(n, weighted, nran):
    case = {"n": n, "box": 1000.0, "assign": L.TSC, "los": False}
    d = cn.mesh_desc(n, 1000.0, assign=L.TSC, interlace=True, dtype=L.F64, observer=cases.OBSERVER)
    (g, gw), (r, rw) = _catalog(max(1, nran // 3), 1), _catalog(nran, 2)
    if not weighted:
        gw = rw = None
    norms, delta, noise, gs, rs = pl.paint_fkp(d, g, r, gw, rw)
    for got, pos, w in ((gs, g, gw), (rs, r, rw)):
        want = cases._sums(case, pos, w)
        # sums of up to 1.3e6 terms of either sign, in any order
        assert bool(((got - want).abs() <= 1e-12 * want[2]).all())
    alpha = norms[L.NORM_ALPHA]
    assert float((alpha - gs[0] / rs[0]).abs()) <= 1e-15 * float(alpha)
    for ph in range(2):
        a, b = cases._paint(case, g, gw, 0.5 * ph), cases._paint(case, r, rw, 0.5 * ph)
        want = a - alpha * b
        # contributions rounded to 2^-40 units, at most nran of them of 27 on a node
        assert float((delta[ph] - want).abs().max()) <= 1e-10 * float((a + alpha * b).max())
        a2, b2 = (cases._paint(case, p, None if w is None else w.double() ** 2, 0.5 * ph) for p, w in ((g, gw), (r, rw)))
        want = a2 + alpha ** 2 * b2
        assert float((noise[ph] - want).abs().max()) <= 1e-10 * float(want.max())
