"""The two kernels of the compiled-length FMT pass (one wave per field on small grids, two waves per
row pair on large ones) at the edges of their tiles: every compiled x length, the last block with
missing row pairs and a missing partner row, FP64, FP32-mixed, the alternative functionals and the
Hessian product, against the oracle.

Tolerances are the bars of the parity tests: FP64 operators 1e-12 of each field's maximum, G of an
FP32-mixed evaluation 5 % away from its reference 1e-6, adjoint weights 1e-5.
"""
import sys

import numpy as np
import pytest
import torch

from oracle import adjoint as oracle_adjoint
from oracle import residual
from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import from_problem
from test_gpu_parity import mixture

pytestmark = pytest.mark.gpu

LENGTHS = [16, 24, 32, 48, 64, 96, 128, 192, 256, 384]
WIDE_BLOCKS = 384     # the launcher's rule: at most so many blocks of 256 // n_x (at least 1) row pairs


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b))) / max(np.max(np.abs(b)), 1e-300))


def _grid(nx, form):
    """(nx, ny, nz): an odd number of rows, and row pairs that do not fill the last block."""
    pw = max(1, 256 // nx)
    if form == "wide":
        return (nx, 9, 27)
    nz = next(n for n in (27, 81, 243) if ((9 * n + 1) // 2 + pw - 1) // pw > WIDE_BLOCKS or n == 243)
    ny = next(n for n in (9, 27, 81) if ((n * nz + 1) // 2 + pw - 1) // pw > WIDE_BLOCKS)
    return (nx, ny, nz)


def _problem(n, functional="rslt", S=2):
    p = mixture(n, h=(0.06, 0.05, 0.055), S=S, es=True, seed=4)
    p.hs_functional = functional
    return p


def _density(p, seed=2, amp=0.3):
    rng = np.random.default_rng(seed)
    return p.initial_density() * (1.0 + amp * rng.uniform(-1.0, 1.0, (p.nspecies,) + p.shape))


@pytest.mark.parametrize("form", ["wide", "paired"])
@pytest.mark.parametrize("nx", LENGTHS)
def test_fields_and_mixed_residual(nx, form):
    p = _problem(_grid(nx, form))
    st = residual.Setup(p)
    rho = _density(p)
    ev = st.evaluate(rho)
    print(f"  {p.n} {form}", file=sys.stderr, flush=True)
    sol = from_problem(p)
    out = sol.operators(_dev(rho))
    for key, ref in (("n", ev["n"]), ("dphi", ev["dphi"])):
        for k in range(10):
            assert _rel(out[key][k].cpu().numpy(), ref[k]) < 1e-12 or np.max(np.abs(ref[k])) < 1e-12, (key, k)
    G, _ = sol.residual(_dev(rho))
    assert _rel(G.cpu().numpy(), ev["G"]) < 1e-12
    sol.close()
    mixed = from_problem(p, precision=_abi.DFT_FP32_MIXED)
    mixed.set_reference(_dev(rho))
    near = _density(p, 3, 0.05) * rho / np.where(rho > 0, p.initial_density(), 1.0)
    G, _ = mixed.residual(_dev(near))
    assert _rel(G.cpu().numpy(), st.G(near)) < 1e-6
    mixed.close()


@pytest.mark.parametrize("functional", ["rosenfeld", "whitebear"])
@pytest.mark.parametrize("nx,form", [(24, "wide"), (24, "paired"), (256, "paired"), (384, "wide")])
def test_alternative_functionals(nx, form, functional):
    p = _problem(_grid(nx, form), functional)
    st = residual.Setup(p)
    rho = _density(p)
    G_ref = st.G(rho)
    for prec, bar in ((_abi.DFT_FP64, 1e-12), (_abi.DFT_FP32_MIXED, 1e-6)):
        sol = from_problem(p, precision=prec)
        sol.set_reference(_dev(p.initial_density() * 0.5 + rho * 0.5))
        G, _ = sol.residual(_dev(rho))
        # FP32 errors are proportional to the distance from the reference (15 % here, 5 % at the bar)
        assert _rel(G.cpu().numpy(), G_ref) < (bar if prec == _abi.DFT_FP64 else 3 * bar)
        sol.close()


@pytest.mark.parametrize("nx,form", [(24, "wide"), (24, "paired"), (128, "paired"), (384, "paired")])
def test_hessian_product(nx, form):
    p = _problem(_grid(nx, form))
    p.rho_bulk = 0.3 * np.asarray(p.rho_bulk)
    st = residual.Setup(p)
    sol = from_problem(p)
    x = _dev(p.initial_density())
    sol.solve(x, 1e-12, 2000)
    g = _dev(np.random.default_rng(1).uniform(0.0, 1.0, (p.nspecies,) + p.shape))
    w = -sol.adjoint(x, g, tol=1e-10)["vext"].cpu().numpy()
    w_ref = oracle_adjoint.adjoint_weights(st, x.cpu().numpy(), g.cpu().numpy(), tol=1e-10)
    w_ref = w_ref[0] if isinstance(w_ref, tuple) else w_ref
    assert _rel(w, w_ref) < 1e-5
    sol.close()
