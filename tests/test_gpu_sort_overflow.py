"""Catalogs that fill a part of their box: most of their records pass the capacity
of the bucket regions and are counted and sorted as overflow records.  The meshes
are integer sums, so with the same normalisations they equal those of the sort with
a histogram pass of its own (CNPC_TUNE_SORT_FUSED 1), which has no capacity, bit for
bit, and painting takes about the time of that sort."""

import contextlib

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402


@contextlib.contextmanager
def sort_fused(v):
    L.check(L.lib.cnpc_tune_set(L.TUNE["sort_fused"][0], v))
    try:
        yield
        torch.cuda.synchronize()
    finally:
        L.check(L.lib.cnpc_tune_set(L.TUNE["sort_fused"][0], 0))


def _catalog(n, box, seed):
    """n particles in the (bx, by, bz) sixteenths of the box from its corner."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.rand((3, n), generator=g, device="cuda", dtype=torch.float64)
    p = (p * torch.tensor(box, device="cuda", dtype=torch.float64)[:, None] * 2.0 ** 28).long()
    return (p - ((p >> 31) << 32)).to(torch.int32), 0.5 + torch.rand(n, generator=g, device="cuda")


# one bucket, 8, 64 and 96 of them (more than a chunk's table holds), whole and
# part chunks; one 16^3 tile
@pytest.mark.parametrize("n,box,nran", [(128, (8, 8, 8), 700_001), (256, (4, 4, 4), 1_000_003), (256, (8, 8, 8), 3_000_017),
                                        (256, (1, 1, 1), 300_007), (512, (2, 2, 2), 900_001), (512, (8, 8, 12), 4_000_037)])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("dtype", [L.F32, L.F64])
def test_overflow_equals_counting_sort(n, box, nran, weighted, dtype):
    d = cn.mesh_desc(n, 1000.0, assign=L.CIC, interlace=False, dtype=dtype)
    (g, gw), (r, rw) = _catalog(nran // 7, box, 1), _catalog(nran, box, 2)
    if not weighted:
        gw = rw = None
    sc = pl.Scratch()
    norms, _, _ = pl.catalog_norms(d, g, r, gw, rw, sc)
    out = {}
    for v in (1, 0):
        with sort_fused(v):
            out[v] = pl.paint(d, g, r, norms, gw, rw, scratch=sc)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def _time(f):
    f()
    ts = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b))
    return min(ts)


@pytest.mark.parametrize("n,box", [(128, (8, 8, 8)), (256, (8, 8, 8)), (256, (4, 4, 4)), (512, (4, 4, 4))])
def test_concentrated_catalog_time(n, box):
    """Measured 0.3 to 1.0 times the counting sort's time; with one global atomic per
    overflow record 4 to 12 at 128 and 256."""
    d = cn.mesh_desc(n, 1000.0, assign=L.TSC, interlace=True, dtype=L.F32)
    m = {128: 2_000_000, 256: 10_000_000, 512: 20_000_000}[n]
    (g, _), (r, _) = _catalog(m // 8, box, 1), _catalog(m, box, 2)
    sc = pl.Scratch()
    norms, _, _ = pl.catalog_norms(d, g, r, None, None, sc)
    t = {}
    for v in (1, 0):
        with sort_fused(v):
            t[v] = _time(lambda: pl.paint(d, g, r, norms, noise=False, scratch=sc))
    assert t[0] < 1.5 * t[1], t
