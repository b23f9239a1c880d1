"""Lengths without compiled kernels (2, 3, 4, 6 and 576 to 1024) on each axis, several stages and ragged tiles: FP64
operators and G against the oracle to 1e-12 of each field's maximum, FP32-mixed G 5 % away from its reference to
1e-6, with the alternative functionals among them (in FP32-mixed the 576 to 768 rows run all ten fields of a row pair
in one block, in FP64 and past 819 one field at a time), more than four charged species, and FP32-mixed with the
screening kernel cut at lambda_i + lambda_j."""
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


def _check(p, seed, cutoff="contact", flags=0):
    st = residual.Setup(p, cutoff)
    # the oracle's 2 - 2 cos(k h) loses digits at long waves (1.8e-12 of it at the first mode of 1024 nodes)
    st.D = sum(4.0 * np.sin(0.5 * st.mesh.comp[d] * p.h[d]) ** 2 / p.h[d] ** 2 for d in range(3))
    rng = np.random.default_rng(seed)
    rho = p.initial_density() * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, (p.nspecies,) + p.shape))
    ev = st.evaluate(rho)
    print(f"  n = {p.n}, S = {p.nspecies}", file=sys.stderr, flush=True)
    sol = from_problem(p, flags=flags)
    assert sol.stats()["compact_layout"] == 0 or flags
    out = sol.operators(_dev(rho))
    for key, ref in (("n", ev["n"]), ("dphi", ev["dphi"]), ("c", ev["E"])):
        for k in range(len(ref)):
            assert _rel(out[key][k].cpu().numpy(), ref[k]) < 1e-12 or np.max(np.abs(ref[k])) < 1e-12, (key, k)
    G, r = sol.residual(_dev(rho))
    assert _rel(G.cpu().numpy(), ev["G"]) < 1e-12
    assert r == pytest.approx(st.residual_norm(st.sqnorm(rho - ev["G"])), rel=1e-12)
    sol.close()
    mixed = from_problem(p, precision=_abi.DFT_FP32_MIXED, flags=flags)
    mixed.set_reference(_dev(rho))
    near = rho * (1.0 + 0.05 * rng.uniform(-1.0, 1.0, rho.shape))
    G, _ = mixed.residual(_dev(near))
    assert _rel(G.cpu().numpy(), st.G(near)) < 1e-6
    mixed.close()


@pytest.mark.parametrize("n,functional",
                         [((576, 6, 9), "rslt"), ((648, 3, 8), "whitebear"), ((768, 8, 3), "rosenfeld"),
                          ((864, 4, 6), "rslt"), ((1024, 3, 4), "whitebear"), ((6, 27, 9), "whitebear"),
                          ((9, 576, 6), "rslt"), ((18, 768, 3), "rslt"), ((4, 972, 8), "rslt"),
                          ((9, 6, 576), "rslt"), ((24, 3, 648), "rslt"), ((16, 4, 1024), "rslt"), ((6, 4, 6), "rosenfeld")])
def test_lengths(n, functional):
    p = mixture(n, h=(0.06, 0.05, 0.055), S=3 if n[1] % 2 else 2, es=True, seed=1)
    p.hs_functional = functional
    _check(p, sum(n))


def _charged(n, S):
    z = np.array([1.0, -1.0, 2.0, -2.0, 1.0, -1.0])[:S]
    rho = np.full(S, 0.2)
    rho[-1] -= (z * rho).sum() / z[-1]
    return W.Problem(name="charged", n=n, h=(0.06, 0.05, 0.055), radius=0.08 + 0.015 * np.arange(S), valence=z,
                     rho_bulk=rho, bjerrum=0.3, electrostatics=True)


@pytest.mark.parametrize("n", [(12, 9, 32), (24, 27, 128), (16, 8, 243)])
def test_more_than_four_charged_species(n):
    _check(_charged(n, 6), 3)


@pytest.mark.parametrize("n", [(24, 9, 32), (16, 24, 128), (27, 8, 243)])
def test_cutoff_at_lambda(n):
    _check(mixture(n, h=(0.06, 0.05, 0.055), S=2, es=True, seed=2), 4, cutoff="lambda", flags=_abi.FLAG_CUTOFF_LAMBDA)
