"""The FP64 Sugiyama contraction forms W in registers: its workspace holds no W fields
and no all-ones field (CPU: sizes only)."""

import ctypes as C
import math

import pytest

import paper_2605_04864_amd as cn
from paper_2605_04864_amd import _lib as L


def _size(n, dtype, cells, nb):
    """Workspace of nb shells up to `cells` fundamental wavenumbers"""
    d = cn.mesh_desc(n, 1000.0, dtype=dtype)
    b = cn.kbins(0.0, cells * 2 * math.pi / 1000.0 / nb, nb)
    return L.lib.cnpc_sugi_workspace_size(C.byref(d), C.byref(b))


def _grid(n, cells, nb):
    """Alias-free grid of two shell fields (|n| < cells) and one of the whole noise band"""
    band = 1
    while band < n // 2 and band <= (2 * nb - 1) * cells / nb:
        band *= 2
    g = 16
    while g < n and (g < 2 * int(cells) + band or g < 2 * band):
        g *= 2
    return g


@pytest.mark.parametrize("nb", [1, 7, 20])
def test_fp64_fields(nb):
    # two grids: the parts that do not grow with the grid cancel
    diff = []
    for n, cells in ((64, 8.5), (256, 30.5)):
        f64, f32, g = _size(n, L.F64, cells, nb), _size(n, L.F32, cells, nb), _grid(n, cells, nb)
        assert f32 > 0 and f64 >= (3 * nb + 2) * g ** 3 * 8
        diff.append(2 * f32 - f64 - (nb + 1) * 8 * g ** 3)
    assert diff[0] == diff[1]
