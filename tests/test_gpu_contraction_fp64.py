"""FP64 contractions (TripoSH, Sugiyama, Scoccimarro) at the edges of their shell tiles
and of the prefetching form, element by element against FP64 sums over the shell fields
that torch's transforms give for the same spectra.  The bar is relative to the size of
each sum's terms, sqrt(sum P_i^2 sum W_j^2): a few FP64 transforms and a sum."""

import ctypes as C

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402
from perf import cases  # noqa: E402
from test_gpu_cross_contraction import _spectra  # noqa: E402

TOL = 1e-12
KF = 2.0 * 3.141592653589793 / 1000.0


class _Modes:
    """Band spectra on the half grid of an n^3 mesh, and shells 1.01 k_f wide."""

    def __init__(self, n, band, nb):
        self.n, self.m = n, band
        self.sh = cases._Shells({"n": n, "box": 1000.0, "dk": 1.01 * KF}, nb)
        self.idx = torch.tensor([j if j < band else j - 2 * band for j in range(2 * band)], device="cuda") % n

    def full(self, spec):
        n, m = self.n, self.m
        out = torch.zeros((n, n, n // 2 + 1), dtype=torch.complex128, device="cuda")
        out[self.idx[:, None], self.idx[None, :], :m] = torch.view_as_complex(spec).reshape(2 * m, 2 * m, m)
        out[n - m] = 0  # the unpaired rows of the band
        out[:, n - m] = 0
        return out

    def real(self, full):
        return torch.fft.irfftn(full, s=(self.n,) * 3, norm="forward").reshape(-1)

    def shells(self, full):
        return torch.stack([self.real(torch.where(self.sh.index == b, full, 0.0)) for b in range(self.sh.nb)])


def _run(plan, call, nout):
    raw, shot, val = (torch.full((nout,), -7.0, dtype=torch.float64, device="cuda") for _ in range(3))
    ws = pl.Scratch().get(plan.ws_bytes)
    L.check(call(raw, shot, val, ws))
    torch.cuda.synchronize()
    return raw


@pytest.mark.parametrize("n,nb", [(32, 1), (32, 2), (128, 15), (128, 16), (128, 17), (128, 31), (256, 32), (256, 33),
                                  (256, 48), (256, 49), (256, 62)])
def test_triposh(n, nb):
    d, bins = cn.mesh_desc(n, 1000.0, dtype=L.F64), cn.kbins(0.0, 1.01 * KF, nb)
    norms = torch.ones(L.NORMS_LEN, dtype=torch.float64, device="cuda")
    plan = pl.BispecPlan(d, bins, L.EST_TRIPOSH, 2, L.PREC_F64, pl.Scratch())
    s = _spectra(n, plan.band, 2, nb)
    raw = _run(plan, lambda r, sh, v, ws: L.lib.cnpc_bispectrum(plan.handle, L.ptr(s[0]), L.ptr(s[1]), None, L.ptr(norms),
                                                               L.ptr(r), L.ptr(sh), L.ptr(v), L.ptr(ws), ws.numel(),
                                                               L.stream_handle()), plan.nconf)
    M = _Modes(n, plan.band, nb)
    P, z = M.shells(M.full(s[0])), M.real(M.full(s[1]))
    W = P * z
    c, size = P @ W.T, torch.sqrt((P * P).sum(1)[:, None] * (W * W).sum(1)[None, :])
    i, j = torch.triu_indices(nb, nb, device="cuda")
    scale = 5.0 / (float(n) ** 3 * M.sh.modes[i] * M.sh.modes[j])
    assert raw.numel() == i.numel()
    assert bool(((raw - scale * c[i, j]).abs() <= TOL * scale * size[i, j]).all())


# up to 40 fields at 128 points a chunk and 26 at 256 wait in registers; 40 shells
@pytest.mark.parametrize("n,ell,nb", [(64, 0, 13), (64, 0, 26), (64, 0, 27), (64, 2, 13), (64, 2, 14), (64, 2, 20),
                                      (64, 2, 21), (128, 0, 40)])
def test_scoccimarro(n, ell, nb):
    d, bins = cn.mesh_desc(n, 1000.0, dtype=L.F64), cn.kbins(0.0, 1.01 * KF, nb)
    norms = torch.ones(L.NORMS_LEN, dtype=torch.float64, device="cuda")
    plan = pl.BispecPlan(d, bins, L.EST_SCOCCIMARRO, ell, L.PREC_F64, pl.Scratch())
    s = _spectra(n, plan.band, 2, nb)
    raw = _run(plan, lambda r, sh, v, ws: L.lib.cnpc_bispectrum(plan.handle, L.ptr(s[0]), L.ptr(s[1]) if ell else None, None,
                                                               L.ptr(norms), L.ptr(r), L.ptr(sh), L.ptr(v), L.ptr(ws),
                                                               ws.numel(), L.stream_handle()), plan.nconf)
    M = _Modes(n, plan.band, nb)
    x = M.shells(M.full(s[0]))
    y = M.shells(M.full(s[1])) if ell else x
    ijk, nt = plan.configs()
    i, j, k = (torch.as_tensor(q, device="cuda").long() for q in ijk.reshape(-1, 3).T.copy())
    nt = torch.as_tensor(nt, device="cuda").double()
    c = torch.stack([(x[a] * x) @ y.T for a in range(nb)])
    size = torch.stack([torch.sqrt(((x[a] * x) ** 2).sum(1)[:, None] * (y * y).sum(1)[None, :]) for a in range(nb)])
    # the l leg is i; the two others in either order
    scale = (2 * ell + 1) / (float(n) ** 3 * nt)
    assert bool(((raw - scale * c[j, k, i]).abs() <= TOL * scale * size[j, k, i]).all())


@pytest.mark.parametrize("l1,l2,lm,nb", [(0, 0, 0, 1), (2, 0, 2, 15), (1, 1, 0, 16), (2, 2, 2, 17), (1, 1, 2, 31)])
def test_sugiyama(l1, l2, lm, nb):
    n = 128
    d, bins = cn.mesh_desc(n, 1000.0, dtype=L.F64, assign=L.TSC), cn.kbins(0.0, 1.01 * KF, nb)
    norms = torch.ones(L.NORMS_LEN, dtype=torch.float64, device="cuda")
    plan = pl.SugiPlan(d, bins, l1, l2, lm, L.PREC_F64)
    s = _spectra(n, plan.band, 2 + 2 * lm, nb)
    raw = _run(plan, lambda r, sh, v, ws: L.lib.cnpc_sugiyama(plan.handle, L.ptr(s[0]), L.ptr(s[1:]) if lm else None, None,
                                                             L.ptr(norms), L.ptr(r), L.ptr(sh), L.ptr(v), L.ptr(ws),
                                                             ws.numel(), L.stream_handle()), nb * nb)
    M = _Modes(n, plan.band, nb)
    f0 = M.full(s[0])
    u = cases._unit(*cases._half(n))
    nx, ny, nz = cases._half(n)
    window = (torch.sinc(nx / n) * torch.sinc(ny / n) * torch.sinc(nz / n)) ** 3
    nyq = (nx.abs() == n // 2) | (ny.abs() == n // 2) | (nz == n // 2)

    def los(q):
        if lm == 0:  # F_0 as it is given, over its window and with what it has at k = 0
            return M.real(f0)
        f = torch.where(nyq, 0.0, M.full(s[1 + q]) / window)
        f[0, 0, 0] = 0
        return M.real(f)

    def pair(l, m):
        return [M.shells(f0 * (1j if l % 2 else 1) * y) for y in cases._ylm(l, abs(m), *u)]

    def both(p, m, l):  # F_l^m = sum conj(y) F_0; odd l: i y F_0 is Hermitian
        re, im = p[0], -p[1] if m >= 0 else p[1]
        sg = (-1) ** m if m < 0 else 1
        return (sg * re, sg * im) if l % 2 == 0 else (sg * im, -sg * re)

    legs = [{m: pair(l, m) for m in range(l + 1)} for l in (l1, l2)]
    c = torch.zeros((nb, nb), device="cuda", dtype=torch.float64)
    size = torch.zeros_like(c)
    for big in range(-lm, lm + 1):
        g = [los(0), torch.zeros(n ** 3, device="cuda", dtype=torch.float64)] if big == 0 else \
            [los(2 * abs(big) - 1), los(2 * abs(big))]
        sg = (-1) ** big if big < 0 else 1
        gr, gi = sg * g[0], -sg * g[1] if big >= 0 else sg * g[1]
        for m1 in range(-l1, l1 + 1):
            m2 = -m1 - big
            w = cases._three_j(l1, l2, lm, m1, m2, big) if abs(m2) <= l2 else 0.0
            if w == 0.0:
                continue
            a, b = both(legs[0][abs(m1)], m1, l1), both(legs[1][abs(m2)], m2, l2)
            for p, v, sign in ((a[0], b[0] * gr - b[1] * gi, 1), (a[1], b[0] * gi + b[1] * gr, -1)):
                c += sign * w * (p @ v.T)
                size += abs(w) * torch.sqrt((p * p).sum(1)[:, None] * (v * v).sum(1)[None, :])
    hn = cases._three_j(l1, l2, lm, 0, 0, 0) * (2 * l1 + 1) * (2 * l2 + 1) * (2 * lm + 1)
    scale = abs(hn) / (float(n) ** 3 * M.sh.modes[:, None] * M.sh.modes[None, :])
    ref = hn / abs(hn) * scale * c
    assert bool(((raw.reshape(nb, nb) - ref).abs() <= TOL * scale * size).all())
