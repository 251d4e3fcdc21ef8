"""Range of the Y_lm transforms: the harmonics of the line of sight depend on no
unit of length, so lengths scaled by a power of two give the same bits; a distant
observer gives the fixed line of sight towards it, and one next to a mesh node the
fields of the oracle's directions."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # the marker deselects these on CPU runs
    pytest.skip("no GPU", allow_module_level=True)

import paper_2605_04864_amd as cn  # noqa: E402
from paper_2605_04864_amd import _lib as L  # noqa: E402
from paper_2605_04864_amd import pipeline as pl  # noqa: E402
from oracle import spectra as osp  # noqa: E402
from oracle.ylm import ylm_racah  # noqa: E402

OBS = np.array([-700.0, -310.0, -1200.0])


def _mesh(n, dtype):
    g = torch.Generator(device="cuda").manual_seed(n)
    return torch.randn((n, n, n), generator=g, dtype=torch.float64, device="cuda").to(pl._TORCH_DT[dtype])


@pytest.mark.parametrize("exp", [40, -48])
@pytest.mark.parametrize("n,band,dtype", [(16, 8, L.F32), (64, 16, L.F32), (128, 32, L.F32), (256, 32, L.F32),
                                          (256, 8, L.F32), (512, 32, L.F32), (128, 32, L.F64)])
def test_ylm_no_unit_of_length(n, band, dtype, exp):
    f = 2.0 ** (exp if dtype == L.F32 else 7 * exp)  # R^4 leaves the range of the type
    x = _mesh(n, dtype)
    ells = (4,) if n == 512 else (1, 2, 3, 4)
    ref = pl.ylm_spectra(cn.mesh_desc(n, 1000.0, dtype=dtype, observer=OBS), band, ells, x)
    got = pl.ylm_spectra(cn.mesh_desc(n, 1000.0 * f, dtype=dtype, observer=OBS * f), band, ells, x)
    for l in ells:
        assert bool(torch.isfinite(ref[l]).all())
        assert torch.equal(got[l], ref[l]), l


@pytest.mark.parametrize("n,band", [(64, 16), (128, 32), (256, 32)])
def test_ylm_distant_observer(n, band):
    """1e10 box lengths away against the fixed direction (1e-10 from it at every
    node); the bar is a few roundings of a row transform and of the sums of up to
    three powers, against the largest value."""
    u = np.array([0.48, 0.6, 0.64])
    x = _mesh(n, L.F32)
    got = pl.ylm_spectra(cn.mesh_desc(n, 1000.0, dtype=L.F32, observer=-1e13 * u), band, (2, 4), x)
    ref = pl.ylm_spectra(cn.mesh_desc(n, 1000.0, dtype=L.F32, los=u), band, (2, 4), x)
    for l in (2, 4):
        assert float((got[l] - ref[l]).abs().max()) < 1e-5 * float(ref[l].abs().max()), l


@pytest.mark.parametrize("off", [1e-13, 1e-9, 0.2])  # in cells
@pytest.mark.parametrize("n,dtype", [(16, L.F64), (64, L.F32), (64, L.F64), (128, L.F32), (128, L.F64), (256, L.F32)])
def test_ylm_observer_at_a_node(n, dtype, off):
    box, band = 1000.0, n // 8
    h = box / n
    obs = np.array([-off * h, 5.0 * h, 3.0 * h])  # beyond the lower x face, beside node (0, 5, 3)
    x = _mesh(n, dtype)
    ells = (2,) if n == 256 else (3, 4)
    got = pl.ylm_spectra(cn.mesh_desc(n, box, dtype=dtype, observer=obs), band, ells, x)
    rvec = osp.line_of_sight(n, box, obs)
    xh = x.double().cpu().numpy()
    idx = np.r_[0:band, n - band:n]
    tol = 2e-9 if dtype == L.F64 else 2e-4
    for l in ells:
        f = 0
        for m in range(l + 1):
            y = ylm_racah(l, m, rvec)
            for w in (y.real,) if m == 0 else (y.real, y.imag):
                ref = np.fft.rfftn(xh * w)[np.ix_(idx, idx, range(band))]
                g = torch.view_as_complex(got[l][f].double()).cpu().numpy().reshape(ref.shape)
                assert np.max(np.abs(g - ref)) < tol * np.max(np.abs(ref)), (l, f)
                f += 1
