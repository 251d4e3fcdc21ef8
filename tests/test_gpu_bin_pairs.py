"""Shell binning of many spectra: every count of pairs and self terms (the kernel
loads four pairs at a time and keeps 4, 8, 12, 16 or 20 sums per thread), bands from
one plane to runs of eight modes, shells that start above k = 0, against FP64 sums
over the modes; and its time, which is to grow with the spectra read, not faster."""

import ctypes as C
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402
from oracle.ylm import ylm_racah  # noqa: E402

KF = 2.0 * math.pi / 1000.0


def _spectra(band, dtype, count):
    g = torch.Generator(device="cuda").manual_seed(band)
    return [torch.randn((pl.band_size(band), 2), generator=g, device="cuda", dtype=torch.float64).to(pl._TORCH_DT[dtype])
            for _ in range(count)]


def _pairs(F, count):
    k = len(F)
    return [(F[i % k], F[(i + 1 + i // k) % k]) for i in range(count)]


def _modes(n, m):
    j = np.arange(2 * m)
    f = np.where(j < m, j, j - 2 * m)
    nx, ny, nz = f[:, None, None], f[None, :, None], np.arange(m)[None, None, :]
    n2 = nx ** 2 + ny ** 2 + nz ** 2
    ok = (n2 > 0) & (nx != -(n // 2)) & (ny != -(n // 2))
    return nx, ny, nz, n2, ok


def _self_value(n, m, assign, interlace, sb, l):
    """Re sum_m y_l^m Sbar_l^m C / W^2 of every mode (closed forms of the alias sums)"""
    nx, ny, nz, n2, _ = _modes(n, m)
    w = c = t = 1.0
    for v in (nx, ny, nz):
        a = v / n
        s2, co = np.sin(math.pi * a) ** 2, np.cos(math.pi * a)
        w = w * np.sinc(a) ** (3 if assign == L.TSC else 2)
        if assign == L.TSC:
            c, t = c * (1 - s2 + 2 / 15 * s2 ** 2), t * co * (co ** 4 + 58 * co ** 2 + 61) / 120
        else:
            c, t = c * (1 - 2 / 3 * s2), t * co * (5 + co ** 2) / 6
    c = 0.5 * (c + t) if interlace else c
    vec = np.stack(np.broadcast_arrays(nx, ny, nz), -1).astype(float)
    base, out = {0: 0, 2: 1, 4: 4}[l], 0.0
    for q in range(l + 1):
        y = ylm_racah(l, q, vec)
        out = out + (1 if q == 0 else 2) * (y.real * sb[2 * (base + q)] - y.imag * sb[2 * (base + q) + 1])
    return out * c / w ** 2


BANDS = [(1, 16, 1, 0.0), (2, 16, 2, 0.0), (8, 16, 5, 1.3), (16, 64, 9, 0.0), (32, 64, 31, 0.0)]
LARGE = [(64, 128, 12, 3.7), (128, 512, 40, 0.0)]
COUNTS = [(3, (0,), False), (9, (), False), (9, (2, 4, 0), False), (16, (4, 2, 0, 2), False), (0, (4,), False)]
MORE = [(1, (), True), (4, (), False), (5, (), False), (4, (0, 2, 4), False), (16, (), True)]


# from band 128 up few pairs with self terms run along kz
@pytest.mark.parametrize("shape,count", [(s, c) for s in BANDS for c in COUNTS + MORE] + [(s, c) for s in LARGE for c in COUNTS]
                         + [(LARGE[1], c) for c in ((1, (2,), False), (2, (0, 4), False))])
@pytest.mark.parametrize("dtype", [L.F32, L.F64])
def test_bin_every_count(shape, count, dtype):
    (band, n, nb, kmin), (npairs, selfs, imag) = shape, count
    assign, il = (L.TSC, 1) if npairs % 2 else (L.CIC, 0)
    d = cn.mesh_desc(n, 1000.0, assign=assign, interlace=bool(il), dtype=dtype)
    top = 0.98 * band if band > 1 else 0.999
    dk = (top - kmin) / nb
    bins = cn.kbins(kmin * KF, dk * KF, nb)
    pairs = _pairs(_spectra(band, dtype, 5), npairs)
    norms = torch.linspace(-0.7, 1.3, L.NORMS_LEN, device="cuda", dtype=torch.float64)
    means, selft, nmodes, keff = pl.bin_means(d, bins, band, pairs, selfs, norms if selfs else None, imag=imag)
    nx, ny, nz, n2, ok = _modes(n, band)
    edges = np.array([math.ceil((kmin + b * dk) ** 2) for b in range(nb + 1)])
    b = np.searchsorted(edges, n2, side="right") - 1
    ok = ok & (b >= 0) & (b < nb)
    wgt = np.broadcast_to(np.where(nz == 0, 1.0, 2.0), n2.shape)[ok]
    idx = b[ok]
    count = np.bincount(idx, wgt, nb)
    assert np.array_equal(nmodes.cpu().numpy(), count.astype(np.int64))
    have = count > 0
    mean = lambda v: (np.bincount(idx, wgt * v[ok], nb)[have] / count[have])
    size = lambda v: (np.bincount(idx, wgt * np.abs(v[ok]), nb)[have] / count[have])
    # FP64 sums over at most 4 m^3 modes in any order
    tol = 1e-13
    assert np.allclose(keff.cpu().numpy()[have], KF * mean(np.sqrt(n2)), rtol=1e-12, atol=0)
    for q, (fa, fb) in enumerate(pairs):
        za, zb = (torch.view_as_complex(x.double()).cpu().numpy().reshape(n2.shape) for x in (fa, fb))
        v = za * zb.conj()
        v = v.imag if imag else v.real
        assert np.all(np.abs(means[q].cpu().numpy()[have] - mean(v)) <= tol * size(v)), q
    sb = norms.cpu().numpy()[L.NORM_SBARLM:]
    for q, l in enumerate(selfs):
        v = _self_value(n, band, assign, il, sb, l)
        assert np.all(np.abs(selft[q].cpu().numpy()[have] - mean(v)) <= 1e-12 * size(v)), q


@pytest.mark.parametrize("band,n", [(128, 512), (256, 512)])
def test_bin_time_of_many_pairs(band, n):
    """FP64, 16 products of four spectra against one product of two: 2.5 times its
    time, 10 with every lane in lines of its own."""
    d = cn.mesh_desc(n, 1000.0, dtype=L.F64)
    bins = cn.kbins(0.0, 0.98 * band * KF / 40, 40)
    F = _spectra(band, L.F64, 4)
    t = {}
    for count in (1, 16):
        f = lambda: pl.bin_means(d, bins, band, _pairs(F, count))
        f()
        ts = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b))
        t[count] = min(ts)
    assert t[16] < 5.0 * t[1], t
