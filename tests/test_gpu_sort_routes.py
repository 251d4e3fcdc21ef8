"""The two sorts of painting on meshes of several tile buckets: the counting sort with a
histogram pass of its own (CNPC_TUNE_SORT_FUSED 1), which cnpc_paint no longer takes by
default, against the oracle in every chunk shape, and the bucket regions against it, bit
for bit on the same normalisations.  Weights of one catalog alone in
cnpc_paint_deinterlace; infinite and NaN weights."""

import contextlib

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import autotune  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402
import test_gpu_parity as P  # noqa: E402


@contextlib.contextmanager
def knobs(**kv):
    autotune.set_knobs(kv)
    try:
        yield
        torch.cuda.synchronize()
    finally:
        autotune.reset_knobs()


# a few buckets, chunks that span many of them, one tile
@pytest.mark.parametrize("threads,per", [(0, 0), (512, 1), (512, 4), (1024, 1), (1024, 2), (1024, 4)])
@pytest.mark.parametrize("case", ["dense128", "sparse256_weighted", "one_tile256"])
def test_counting_sort_vs_oracle(case, threads, per):
    with knobs(sort_fused=1, sort_threads=threads, sort_per=per):
        P.test_paint_bucketed_sort(case)


@pytest.mark.parametrize("weights", [False, True])
def test_counting_sort_of_a_concentrated_catalog(weights):
    g, gw, r, rw, ora, od, onm = P._overflow_case(weights)
    d = cn.mesh_desc(256, 1000.0, assign=L.TSC, interlace=True, dtype=L.F32, observer=P.OBS)
    gt, rt = P.dev(g), P.dev(r)
    gwt, rwt = (P.dev(gw), P.dev(rw)) if weights else (None, None)
    norms, _, _ = pl.catalog_norms(d, gt, rt, gwt, rwt)
    with knobs(sort_fused=1):
        delta, nmesh = pl.paint(d, gt, rt, norms, gwt, rwt)
    for ph in range(2):
        assert P.rel(P.host(delta)[ph], od[ph]) < 20 * P.TOL[L.F32]
        assert P.rel(P.host(nmesh)[ph], onm[ph]) < 20 * P.TOL[L.F32]
    for bucket in (0, 1, 2, 3):
        with knobs(bucket=bucket):
            delta2, nmesh2 = pl.paint(d, gt, rt, norms, gwt, rwt)
        assert torch.equal(delta, delta2) and torch.equal(nmesh, nmesh2)


def _catalog(n, dense, seed):
    """n particles, half the box along x holding the share `dense` of them."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.randint(0, 1 << 32, (3, n), generator=g, device="cuda", dtype=torch.int64)
    low = torch.rand(n, generator=g, device="cuda") < dense
    p[0] = (p[0] >> 1) + torch.where(low, 0, 1 << 31)
    return (p - ((p >> 31) << 32)).to(torch.int32), 0.5 + torch.rand(n, generator=g, device="cuda")


# 512: 8-byte, 12-byte and 16-byte region records; regions of 1.2 chunks of the
# histogram (7.4e4 of at most 8.1e4 records) beside ones of 0.4.  1024: 4096 buckets
@pytest.mark.parametrize("n,nran,dtype,weighted", [(512, 25_000_001, L.F32, False), (512, 25_000_001, L.F64, False),
                                                   (512, 25_000_001, L.F32, True), (1024, 3_000_001, L.F32, False),
                                                   (1024, 3_000_001, L.F32, True)])
def test_region_histogram(n, nran, dtype, weighted):
    d = cn.mesh_desc(n, 2000.0, assign=L.CIC, interlace=False, dtype=dtype)
    (g, gw), (r, rw) = _catalog(nran // 8, 0.5, 1), _catalog(nran, 0.75, 2)
    if not weighted:
        gw = rw = None
    norms, _, _ = pl.catalog_norms(d, g, r, gw, rw)
    out = {}
    for v in (1, 0):
        with knobs(sort_fused=v):
            out[v] = pl.paint(d, g, r, norms, gw, rw, scratch=pl.Scratch())
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("sort_fused", [0, 1])
@pytest.mark.parametrize("dtype", [L.F32, L.F64])
@pytest.mark.parametrize("side", ["galaxies", "randoms"])
def test_weights_of_one_catalog(side, dtype, sort_fused):
    """cnpc_paint_deinterlace with weights for one catalog only equals weights of one
    for the other (FP32: up to the records' 2^-17 cell grid and 2^-21 units of the
    unit-weight painter)."""
    d = cn.mesh_desc(256, 1000.0, assign=L.TSC, interlace=True, dtype=dtype, observer=P.OBS)
    (g, gw), (r, rw) = _catalog(30_000, 0.5, 3), _catalog(200_001, 0.5, 4)
    one = torch.ones(r.shape[1] if side == "galaxies" else g.shape[1], device="cuda")
    with knobs(sort_fused=sort_fused):
        if side == "galaxies":
            a, b = pl.paint_deinterlace(d, 64, g, r, gw, None), pl.paint_deinterlace(d, 64, g, r, gw, one)
        else:
            a, b = pl.paint_deinterlace(d, 64, g, r, None, rw), pl.paint_deinterlace(d, 64, g, r, one, rw)
    tol = 1e-12 if dtype == L.F64 else 1e-5
    for x, y in zip(a[:4], b[:4]):
        assert float((x - y).abs().max()) <= tol * float(y.abs().max())


@pytest.mark.parametrize("dtype", [L.F32, L.F64])
@pytest.mark.parametrize("n", [64, 128])
def test_infinite_and_nan_weights_stay_on_their_nodes(n, dtype):
    """On fixed normalisations a particle of infinite, NaN or huge weight changes no
    node outside its own stencil."""
    d = cn.mesh_desc(n, 1000.0, assign=L.TSC, interlace=True, dtype=dtype)
    (g, gw), (r, rw) = _catalog(3000, 0.5, 5), _catalog(20_000, 0.5, 6)
    norms, _, _ = pl.catalog_norms(d, g, r, gw, rw)
    bad = {11: float("inf"), 500: float("nan"), 1200: -float("inf"), 2999: 3e38}
    w0, w1 = gw.clone(), gw.clone()
    for i, v in bad.items():
        w0[i], w1[i] = 0.0, v
    ref = pl.paint(d, g, r, norms, w0, rw)
    got = pl.paint(d, g, r, norms, w1, rw)
    base = (g[:, list(bad)].cpu().numpy().astype(np.int64) & 0xFFFFFFFF) >> (32 - int(np.log2(n)))
    own = torch.zeros((n, n, n), dtype=torch.bool, device="cuda")
    for q in range(base.shape[1]):
        i = [torch.tensor([(int(base[a, q]) + o) % n for o in (-1, 0, 1, 2)], device="cuda") for a in range(3)]
        own[i[0][:, None, None], i[1][None, :, None], i[2][None, None, :]] = True
    for x, y in zip(got, ref):
        for ph in range(2):
            assert torch.equal(x[ph][~own], y[ph][~own])
            assert not torch.equal(x[ph][own], y[ph][own])
