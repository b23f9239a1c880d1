"""Conjugate gradients where the system is not positive definite (p.q < 0 in the first iteration, as in the
oracle's operator): the adjoint reports it, Newton keeps the direction it has, and both write no step."""
import numpy as np
import pytest
import torch

from oracle import adjoint as oadj
from oracle import residual
from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import from_problem
from test_gpu_parity import mixture

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.filterwarnings("ignore")
def test_strong_coupling():
    p = mixture((12, 9, 16), h=(0.06, 0.05, 0.055), S=2, es=True, seed=3)
    p.bjerrum = 2.0
    st = residual.Setup(p)
    rho = p.initial_density()
    G = np.asarray(st.evaluate(rho)["G"])
    fluid = G > 0
    g = np.where(fluid, np.array([1.0, -1.0]).reshape(2, 1, 1, 1), 0.0)
    d = G * np.where(fluid, oadj.hessian_vec(st, rho, G * g), 0.0)
    q = np.where(fluid, d / np.where(fluid, G, 1.0) - oadj.hessian_vec(st, rho, d), 0.0)
    assert np.sum(d * q) < 0.0
    sol = from_problem(p)
    with pytest.raises(_abi.DftError, match="not positive definite"):
        sol.adjoint(_dev(rho), _dev(g))
    x = _dev(rho)
    sol.newton(x, 1e-10, 3, raise_on_fail=False)
    x = x.cpu().numpy()
    assert np.all(np.isfinite(x)) and np.all(x >= 0.0)
    sol.close()
