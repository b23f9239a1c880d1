"""Both kernels of the z passes (one wave per transform on small grids, one block per tile above) where the
other length tests run only one of them: the small-grid kernel in the tuned lengths, in both layouts of the
vector densities and with one to five species, and the tiles of the lengths compiled in one shape.  Against
the oracle: FP64 operators to 1e-12 of each field's maximum, FP32-mixed G 5 % away from its reference to 1e-6
(the bars of the parity tests)."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from oracle import residual
from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import from_problem
from test_gpu_parity import mixture

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b))) / max(np.max(np.abs(b)), 1e-300))


def _check(p, seed):
    st = residual.Setup(p)
    rng = np.random.default_rng(seed)
    rho = p.initial_density() * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, (p.nspecies,) + p.shape))
    ev = st.evaluate(rho)
    print(f"  n = {p.n}, S = {p.nspecies}", file=sys.stderr, flush=True)
    sol = from_problem(p)
    out = sol.operators(_dev(rho))
    for k in range(10):
        ref = ev["n"][k]
        assert _rel(out["n"][k].cpu().numpy(), ref) < 1e-12 or np.max(np.abs(ref)) < 1e-12, k
    assert _rel(out["c"].cpu().numpy(), ev["E"]) < 1e-12
    sol.close()
    mixed = from_problem(p, precision=_abi.DFT_FP32_MIXED)
    mixed.set_reference(_dev(rho))
    near = rho * (1.0 + 0.05 * rng.uniform(-1.0, 1.0, rho.shape))
    G, _ = mixed.residual(_dev(near))
    assert _rel(G.cpu().numpy(), st.G(near)) < 1e-6
    mixed.close()


@pytest.mark.parametrize("nx", [24, 18])   # compact vector layout, ten spectra
@pytest.mark.parametrize("length", [16, 24, 32, 48, 64, 96, 128, 192, 256])
def test_small_grids_of_the_tuned_lengths(length, nx):
    _check(mixture((nx, 9, length), h=(0.06, 0.05, 0.055), S=3 if length % 3 else 2, es=True, seed=length), length)


@pytest.mark.parametrize("S,es", [(1, False), (5, False), (8, False), (4, True)])
def test_species_counts(S, es):
    n = (24, 9, 32)
    rho = np.linspace(0.2, 0.5, S)
    z = np.zeros(S)
    if es:
        z = np.array([1.0, -1.0, 2.0, -2.0])
        rho = np.array([0.4, 0.4, 0.2, 0.2])
    p = W.Problem(name="species", n=n, h=(0.06, 0.05, 0.055), radius=0.08 + 0.015 * np.arange(S), valence=z, rho_bulk=rho,
                  bjerrum=0.3 if es else 0.0, electrostatics=es)
    _check(p, S)


@pytest.mark.parametrize("length", [8, 9, 12, 18, 27, 36, 54, 72, 81, 108, 144, 162, 216, 243, 288, 324, 432, 486, 512])
def test_tiles_of_the_one_shape_lengths(length):
    nx, ny = (64, 81) if length <= 64 else (48, 64) if length <= 96 else (32, 64)
    _check(mixture((nx, ny, length), h=(0.06, 0.05, 0.055), S=2, es=True, seed=length), length)
