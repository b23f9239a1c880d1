"""Launch shapes of the z passes on grids past the limits of the small-grid kernels, which have none: in every tuned z
length, each tile width of Z1 (fused, and split from the plain z pass) and of Z2 gives the residual of the default
shape bit for bit, and that one the oracle's (FP64 1e-12, FP32-mixed 5 % from its reference 1e-6).  On small grids
the autotuner has nothing to choose and the schedule says so."""
import sys

import numpy as np
import pytest
import torch

from oracle import residual
from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import from_problem
from test_gpu_parity import mixture
from test_gpu_tune import NSHAPE

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b))) / max(np.max(np.abs(b)), 1e-300))


def _grid(length):
    """(nx, ny, length) whose blocks of four columns exceed every limit of the small-grid kernels."""
    nx, ny, limit = (96, 96, 1100) if length <= 48 else (64, 96, 640) if length <= 96 else (32, 72, 256)
    assert -(-ny * (nx // 2 + 1) // 4) > limit
    return (nx, ny, length)


@pytest.mark.parametrize("S,es", [(2, True), (3, True), (2, False)])
@pytest.mark.parametrize("length", [16, 24, 32, 48, 64, 96, 128, 192, 256, 384])
def test_every_shape_past_the_small_grids(length, S, es):
    p = mixture(_grid(length), h=(0.06, 0.05, 0.055), S=S, es=es, seed=length)
    st = residual.Setup(p)
    rng = np.random.default_rng(length)
    rho = p.initial_density() * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, (S,) + p.shape))
    near = rho * (1.0 + 0.05 * rng.uniform(-1.0, 1.0, rho.shape))
    G_ref = st.G(near)
    print(f"  {p.n} S = {S} es = {es}", file=sys.stderr, flush=True)
    for t, (precision, bar) in enumerate(((_abi.DFT_FP64, 1e-12), (_abi.DFT_FP32_MIXED, 1e-6))):
        sol = from_problem(p, precision=precision, flags=_abi.FLAG_NO_AUTOTUNE)
        if t:
            sol.set_reference(_dev(rho))
        x = _dev(near)
        g0, r0 = sol.residual(x)
        g0 = g0.clone()
        assert _rel(g0.cpu().numpy(), G_ref) < bar
        for name in ("z_weights", "z_back"):
            for v in range(1, NSHAPE[name]):
                sched = {k: (0, 0) for k in NSHAPE}
                sched[name] = (0, v) if t else (v, 0)
                sol.set_schedule(sched)
                g, r = sol.residual(x)
                assert torch.equal(g, g0) and r == r0, (name, v, precision)
        sol.close()


@pytest.mark.parametrize("n", [(24, 24, 24), (48, 48, 48), (32, 32, 96)])
def test_nothing_to_tune_on_small_grids(n):
    sol = from_problem(mixture(n), precision=_abi.DFT_FP32_MIXED)
    s = sol.schedule()
    assert s["z_weights"] == (0, 0) and s["z_back"] == (0, 0)
    # a saved schedule of such a grid may name any shape
    sol.set_schedule(dict(s, z_weights=(5, 5), z_back=(2, 2)))
    sol.close()
