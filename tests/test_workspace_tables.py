"""Workspace of the spectral tables: rows are even in k_z and hold z <= n_z / 2 only, in whole 4 KB (host-only check)."""
import ctypes

import pytest

import workloads as W
from paper_0910_1531_amd import _abi
from test_abi_host import _params


def _size(p):
    n = ctypes.c_size_t()
    assert _abi.load().dft_workspace_size(ctypes.byref(p), ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("n", [(64, 32, 96), (24, 18, 81)])   # even and odd compiled z lengths
def test_rows_hold_half_of_the_planes(n):
    prob = W.charged_sphere(n=n, h=0.1, sigma=(0.3, 0.24), conc=(0.5, 0.5), sphere_radius=0.3)
    es, hs = _params(prob), _params(prob)
    hs.electrostatics = 0
    row = 4096 * -(-8 * (n[2] // 2 + 1) * n[1] * (n[0] // 2 + 1) // 4096)
    # two species: the three pair rows come with electrostatics (buffers are aligned to 256 bytes)
    assert abs(_size(es) - _size(hs) - 3 * row) <= 256
