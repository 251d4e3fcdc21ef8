"""Painting on meshes of more tiles than a workgroup counts in LDS (512^3).

The tile histogram then comes from the bucket-sorted records instead of the
catalog; the meshes are integer sums, so they equal those of the sort with a
histogram pass of its own (CNPC_TUNE_SORT_FUSED 1, which is pinned to the oracle
on smaller meshes) bit for bit, for uniform catalogs and for clustered ones
whose records overflow their bucket regions.
"""

import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402
import test_gpu_parity as P  # noqa: E402


def _catalog(n, clustered, seed):
    rng = np.random.default_rng(seed)
    p = rng.integers(0, 1 << 32, (3, n), dtype=np.uint64)
    if clustered:  # three quarters of the particles in one bucket's corner of the box
        p[:, : 3 * n // 4] >>= 4
    w = rng.uniform(0.5, 1.5, n).astype(np.float32)
    return torch.from_numpy(p.astype(np.uint32)).cuda(), torch.from_numpy(w).cuda()


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("dtype", [L.F32, L.F64])
def test_paint_512_matches_histogram_pass(dtype, weighted, clustered):
    d = cn.mesh_desc(512, 2000.0, assign=L.TSC, interlace=True, dtype=dtype)
    g, gw = _catalog(40_001, clustered, 5)
    r, rw = _catalog(400_003, clustered, 6)
    if not weighted:
        gw = rw = None
    sc = pl.Scratch()
    out = {}
    for knob in (1, 0):
        L.check(L.lib.cnpc_tune_set(L.TUNE["sort_fused"][0], knob))
        try:
            norms, delta, noise, gs, rs = pl.paint_fkp(d, g, r, gw, rw, scratch=sc)
            delta2, noise2 = pl.paint(d, g, r, norms, gw, rw, scratch=sc)
            torch.cuda.synchronize()
        finally:
            L.check(L.lib.cnpc_tune_set(L.TUNE["sort_fused"][0], 0))
        assert torch.equal(delta, delta2) and torch.equal(noise, noise2)
        out[knob] = (norms, delta, noise)
    # the catalog sums run in another order: alpha to a few ulp, and with it the meshes
    tol = 1e-13 if dtype == L.F64 else 2.0 ** -22
    for a, b in zip(out[0], out[1]):
        scale = float(b.abs().max())
        assert float((a - b).abs().max()) <= tol * scale


@pytest.mark.parametrize("dtype,band", [(L.F32, 0), (L.F64, 128)])
def test_fft_512_both_directions(dtype, band):
    """512^3 transforms (z passes of one wavefront per row pair) against numpy, the
    full half spectrum and a band of two kz per lane."""
    n, m = 512, band or 256
    d = cn.mesh_desc(n, 100.0, dtype=dtype)
    tdt = torch.float64 if dtype == L.F64 else torch.float32
    x = np.random.default_rng(band).normal(size=(n, n, n)).astype(np.float32)
    ref = np.fft.rfftn(x.astype(np.float64))
    idx = np.r_[0:m, n - m:n] if band else np.arange(n)
    ref = np.ascontiguousarray(ref[:, :, :m] if not band else ref[np.ix_(idx, idx, range(m))])
    xt = torch.from_numpy(x).to(tdt).cuda()
    spec = torch.empty(ref.shape + (2,), dtype=tdt, device="cuda")
    ws = torch.empty(max(256, L.lib.cnpc_fft_workspace_size(C.byref(d), 1, band)), dtype=torch.uint8, device="cuda")
    L.check(L.lib.cnpc_fft_r2c(C.byref(d), 1, band, L.ptr(xt), L.ptr(spec), L.ptr(ws), ws.numel(), L.stream_handle()))
    got = torch.view_as_complex(spec.double()).cpu().numpy()
    tol = 1e-10 if dtype == L.F64 else 1e-5
    assert np.max(np.abs(got - ref)) < tol * np.max(np.abs(ref))
    # back: the band's modes alone, the Nyquist / n = -m rows empty
    ref[m if band else n // 2] = 0
    ref[:, m if band else n // 2] = 0
    full = np.zeros((n, n, n // 2 + 1), dtype=np.complex128)
    full[np.ix_(idx, idx, range(m))] = ref
    want = np.fft.irfftn(full, s=(n, n, n), axes=(0, 1, 2)) * float(n) ** 3
    st = torch.view_as_real(torch.from_numpy(ref)).to(tdt).cuda().contiguous()
    mesh = torch.empty((n, n, n), dtype=tdt, device="cuda")
    L.check(L.lib.cnpc_fft_c2r(C.byref(d), 1, band, L.ptr(st), L.ptr(mesh), L.ptr(ws), ws.numel(), L.stream_handle()))
    assert np.max(np.abs(mesh.double().cpu().numpy() - want)) < tol * np.max(np.abs(want))


# the z pass in lane groups: one, two and four kz per lane, odd and even l
# together, a global line of sight
@pytest.mark.parametrize("n,band,dtype,ells,los", [
    (64, 8, L.F64, (1, 2, 3, 4), None), (64, 32, L.F64, (4,), None), (128, 16, L.F32, (1, 3), None),
    (128, 64, L.F64, (2,), None), (256, 64, L.F64, (1, 2, 3, 4), None), (128, 32, L.F64, (2, 4), P.YLM_LOS)])
def test_ylm_lane_groups(n, band, dtype, ells, los):
    P.test_ylm_r2c_band(n, band, dtype, ells, los)


@pytest.mark.parametrize("dtype,tol", [(L.F32, 2e-5), (L.F64, 1e-10)])
def test_ylm_512_matches_field_transforms(dtype, tol):
    """512^3: fields from the powers of r_z against one transform per field
    (CNPC_TUNE_YLM_BASIS 1)."""
    d = cn.mesh_desc(512, 2000.0, dtype=dtype)
    x = torch.randn((512, 512, 512), dtype=torch.float64, device="cuda").to(pl._TORCH_DT[dtype])
    out = {}
    for knob in (0, 1):
        L.check(L.lib.cnpc_tune_set(L.TUNE["ylm_basis"][0], knob))
        try:
            out[knob] = pl.ylm_spectra(d, 128, (2,), x)[2]
            torch.cuda.synchronize()
        finally:
            L.check(L.lib.cnpc_tune_set(L.TUNE["ylm_basis"][0], 0))
    for a, b in zip(out[0], out[1]):
        assert float((a - b).abs().max()) <= tol * float(b.abs().max())


@pytest.mark.parametrize("dtype,tol", [(L.F32, 1e-6), (L.F64, 1e-12)])
@pytest.mark.parametrize("n,assign", [(16, L.TSC), (16, L.CIC), (64, L.TSC), (64, L.CIC)])
def test_paint_weights_beyond_the_mantissa_range(n, assign, dtype, tol):
    """Weights of both signs below and above 1024 (w^2 up to 4e6): contributions
    past 2^51 units take the 64-bit conversion, the others the mantissa."""
    from oracle import mesh as oms
    rng = np.random.default_rng(3)
    cat = []
    for k, m in enumerate((1501, 4099)):
        w = np.where(rng.uniform(size=m) < 0.5, rng.uniform(0.5, 2.0, m), rng.uniform(900.0, 2000.0, m))
        w = (w * np.where(rng.uniform(size=m) < 0.2, -1.0, 1.0)).astype(np.float32)
        cat += [rng.integers(0, 1 << 32, (3, m), dtype=np.uint64).astype(np.uint32), w]
    g, gw, r, rw = cat
    d = cn.mesh_desc(n, 300.0, assign=assign, interlace=True, dtype=dtype)
    dev = [torch.from_numpy(x).cuda() for x in cat]
    norms, delta, noise, _, _ = pl.paint_fkp(d, dev[0], dev[2], dev[1], dev[3])
    alpha = float(norms[L.NORM_ALPHA])
    od, on = oms.paint_fkp(g, gw, r, rw, alpha, n, assign, True)
    for got, ref in ((delta, od), (noise, on)):
        for ph in range(2):
            e = np.abs(got[ph].double().cpu().numpy() - ref[ph])
            assert np.max(e) <= tol * np.max(np.abs(ref[ph]))


@pytest.mark.parametrize("n,band,dtype", [(128, 64, L.F32), (128, 16, L.F64), (256, 32, L.F64), (512, 64, L.F32), (512, 128, L.F64)])
def test_deinterlace_fused_x_pass(n, band, dtype):
    """The fused x pass of 128, FP64 256 and 512 (both phases forward, combination, band
    copy, inverse) against the plain passes (CNPC_TUNE_FFT_PASSES 1)."""
    d = cn.mesh_desc(n, 1000.0, interlace=True, dtype=dtype)
    x = torch.randn((2, n, n, n), dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(n)).to(pl._TORCH_DT[dtype])
    out = {}
    for knob in (0, 1):
        L.check(L.lib.cnpc_tune_set(L.TUNE["fft_passes"][0], knob))
        try:
            out[knob] = pl.deinterlace(d, band, x)
            torch.cuda.synchronize()
        finally:
            L.check(L.lib.cnpc_tune_set(L.TUNE["fft_passes"][0], 0))
    tol = 1e-12 if dtype == L.F64 else 2e-6
    for a, b in zip(out[0], out[1]):
        assert float((a - b).abs().max()) <= tol * float(b.abs().max())


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("dtype", [L.F32, L.F64])
@pytest.mark.parametrize("n", [256, 512])
def test_fold_rows_exact_on_nodes(n, dtype, weighted):
    """Row fold on a sparse catalog of particles exactly on nodes, at tile faces and
    the box's periodic faces, with weights of powers of two and alpha = 1: every
    contribution is a multiple of 2^-13, so both meshes are exact in either type."""
    d = cn.mesh_desc(n, 2000.0, assign=L.TSC, interlace=True, dtype=dtype)
    shift = 32 - int(np.log2(n))
    rng = np.random.default_rng(9)
    faces = np.array([0, 1, 14, 15, 16, 17, n // 2 - 1, n // 2, n - 17, n - 16, n - 2, n - 1])
    m = 900
    w = rng.choice(np.array([0.5, 1.0, 2.0], dtype=np.float32), m)
    cat = [((rng.choice(faces, (3, m)).astype(np.uint64)) << np.uint64(shift)).astype(np.uint32) for _ in range(2)]
    g, r = (torch.from_numpy(x).cuda() for x in cat)
    wt = (torch.from_numpy(w).cuda(), torch.from_numpy(w[::-1].copy()).cuda()) if weighted else (None, None)
    norms, delta, nmesh, _, _ = pl.paint_fkp(d, g, r, *wt)
    assert float(norms[L.NORM_ALPHA]) == 1.0
    # TSC of a particle on node c: phase A nodes c - 1 .. c + 1; phase B (u - 1/2) nodes c - 1, c
    sten = (((-1, 0.125), (0, 0.75), (1, 0.125)), ((-1, 0.5), (0, 0.5)))
    for ph in range(2):
        ref = torch.zeros((2, n ** 3), dtype=torch.float64, device="cuda")
        for pos, ww, sign in ((cat[0], wt[0], 1.0), (cat[1], wt[1], -1.0)):
            c = torch.from_numpy((pos >> shift).astype(np.int64)).cuda()
            ww = ww.double() if weighted else torch.ones(m, dtype=torch.float64, device="cuda")
            for ox, vx in sten[ph]:
                for oy, vy in sten[ph]:
                    for oz, vz in sten[ph]:
                        idx = (((c[0] + ox) % n) * n + (c[1] + oy) % n) * n + (c[2] + oz) % n
                        ref[0].index_add_(0, idx, sign * ww * (vx * vy * vz))
                        ref[1].index_add_(0, idx, ww * ww * (vx * vy * vz))
        assert torch.equal(delta[ph].reshape(-1).double(), ref[0])
        assert torch.equal(nmesh[ph].reshape(-1).double(), ref[1])
