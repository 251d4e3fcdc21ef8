"""FP64 shell-by-shell contractions (TripoSH and Sugiyama) at the edges of their
16-shell tiles, against the FP32 path, whose contractions take a row per shell
pair and are pinned to the oracle elsewhere: the same spectra in both types,
within the FP32 bar."""

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


def _spectra(n, band, count, seed):
    """`count` band spectra of white noise on an n^3 mesh (FP64)."""
    d = cn.mesh_desc(n, 1000.0, dtype=L.F64)
    x = torch.randn((count, n, n, n), dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(seed))
    out = torch.empty((count, pl.band_size(band), 2), dtype=torch.float64, device="cuda")
    ws = torch.empty(L.lib.cnpc_fft_workspace_size(C.byref(d), count, band), dtype=torch.uint8, device="cuda")
    L.check(L.lib.cnpc_fft_r2c(C.byref(d), count, band, L.ptr(x), L.ptr(out), L.ptr(ws), ws.numel(),
                               L.stream_handle()))
    return out


def _both(n, nb, make_plan, call, count):
    kf = 2.0 * np.pi / 1000.0
    bins = cn.kbins(0.0, 1.01 * kf, nb)
    norms = torch.ones(L.NORMS_LEN, dtype=torch.float64, device="cuda")
    res = {}
    for dt, prec in ((L.F64, L.PREC_F64), (L.F32, L.PREC_F32)):
        d = cn.mesh_desc(n, 1000.0, dtype=dt)
        sc = pl.Scratch()
        plan = make_plan(d, bins, prec, sc)
        spec = _spectra(n, plan.band, count, nb).to(pl._TORCH_DT[dt]).contiguous()
        raw, shot, val = (torch.full((nb * nb,), -7.0, dtype=torch.float64, device="cuda") for _ in range(3))
        ws = sc.get(plan.ws_bytes)
        call(plan, spec, norms, raw, shot, val, ws)
        torch.cuda.synchronize()
        res[dt] = raw.cpu().numpy()
    assert np.all(np.isfinite(res[L.F64]))
    assert np.max(np.abs(res[L.F32] - res[L.F64])) < 1e-5 * np.max(np.abs(res[L.F64]))


@pytest.mark.parametrize("n,nb", [(32, 1), (128, 15), (128, 16), (128, 17), (256, 33), (256, 49), (256, 62)])
def test_triposh_tiles(n, nb):
    def call(plan, s, norms, raw, shot, val, ws):
        L.check(L.lib.cnpc_bispectrum(plan.handle, L.ptr(s[0]), L.ptr(s[1]), None, L.ptr(norms), L.ptr(raw), L.ptr(shot),
                                      L.ptr(val), L.ptr(ws), ws.numel(), L.stream_handle()))
    _both(n, nb, lambda d, b, p, sc: pl.BispecPlan(d, b, L.EST_TRIPOSH, 2, p, sc), call, 2)


@pytest.mark.parametrize("l1,l2,lm,nb", [(2, 0, 2, 15), (1, 1, 0, 16), (2, 2, 2, 17), (1, 1, 2, 31)])
def test_sugiyama_tiles(l1, l2, lm, nb):
    def call(plan, s, norms, raw, shot, val, ws):
        L.check(L.lib.cnpc_sugiyama(plan.handle, L.ptr(s[0]), L.ptr(s[1:]) if lm else None, None, L.ptr(norms),
                                    L.ptr(raw), L.ptr(shot), L.ptr(val), L.ptr(ws), ws.numel(), L.stream_handle()))
    _both(128, nb, lambda d, b, p, sc: pl.SugiPlan(d, b, l1, l2, lm, p), call, 1 + 2 * lm + 1)


# FP64 row-per-pair contraction with the next chunk in registers (up to 40 fields
# at 128 points a chunk, 26 at 256) and without (more fields)
@pytest.mark.parametrize("ell,nb", [(0, 13), (0, 26), (2, 13), (2, 14), (2, 20), (2, 21)])
def test_scoccimarro_prefetch_edges(ell, nb):
    kf = 2.0 * np.pi / 1000.0
    bins = cn.kbins(0.0, 1.01 * kf, nb)
    norms = torch.ones(L.NORMS_LEN, dtype=torch.float64, device="cuda")
    res = {}
    for dt, prec in ((L.F64, L.PREC_F64), (L.F32, L.PREC_F32)):
        d = cn.mesh_desc(64, 1000.0, dtype=dt)
        sc = pl.Scratch()
        plan = pl.BispecPlan(d, bins, L.EST_SCOCCIMARRO, ell, prec, sc)
        s = _spectra(64, plan.band, 2, nb).to(pl._TORCH_DT[dt]).contiguous()
        raw, shot, val = (torch.zeros(plan.nconf, dtype=torch.float64, device="cuda") for _ in range(3))
        ws = sc.get(plan.ws_bytes)
        L.check(L.lib.cnpc_bispectrum(plan.handle, L.ptr(s[0]), L.ptr(s[1]) if ell else None, None, L.ptr(norms),
                                      L.ptr(raw), L.ptr(shot), L.ptr(val), L.ptr(ws), ws.numel(), L.stream_handle()))
        torch.cuda.synchronize()
        res[dt] = raw.cpu().numpy()
    assert np.max(np.abs(res[L.F32] - res[L.F64])) < 1e-5 * np.max(np.abs(res[L.F64]))
