"""The transform lengths compiled in one launch shape, on every axis, against the oracle: odd row counts,
tiles that cross rows and a partial last tile.  FP64 operators to 1e-12 of each field's maximum, G of an
FP32-mixed evaluation 5 % away from its reference to 1e-6 (the bars of the parity tests)."""
import sys

import numpy as np
import pytest
import torch

from oracle import residual
from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import from_problem
from test_gpu_parity import mixture

pytestmark = pytest.mark.gpu

LENGTHS = [8, 9, 12, 18, 27, 36, 54, 72, 81, 108, 144, 162, 216, 243, 288, 324, 432, 486, 512]


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b))) / max(np.max(np.abs(b)), 1e-300))


@pytest.mark.parametrize("axis", ["x", "y", "z"])
@pytest.mark.parametrize("length", LENGTHS)
def test_length(length, axis):
    n = {"x": (length, 9, 27), "y": (16, length, 27), "z": (24, 9, length)}[axis]
    p = mixture(n, h=(0.06, 0.05, 0.055), S=3 if length % 2 else 2, es=True, seed=length)
    st = residual.Setup(p)
    rng = np.random.default_rng(length)
    rho = p.initial_density() * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, (p.nspecies,) + p.shape))
    ev = st.evaluate(rho)
    print(f"  n = {n}", file=sys.stderr, flush=True)
    sol = from_problem(p)
    assert sol.stats()["compact_layout"] == (0 if axis == "x" and length in (8, 9, 12, 18) else 1)
    out = sol.operators(_dev(rho))
    for key, ref in (("n", ev["n"]), ("dphi", ev["dphi"]), ("c", ev["E"])):
        for k in range(len(ref)):
            assert _rel(out[key][k].cpu().numpy(), ref[k]) < 1e-12 or np.max(np.abs(ref[k])) < 1e-12, (key, k)
    assert _rel(out["phi"].cpu().numpy(), ev["phi"]) < 1e-12
    G, r = sol.residual(_dev(rho))
    assert _rel(G.cpu().numpy(), ev["G"]) < 1e-12
    assert r == pytest.approx(st.residual_norm(st.sqnorm(rho - ev["G"])), rel=1e-12)
    sol.close()
    mixed = from_problem(p, precision=_abi.DFT_FP32_MIXED)
    mixed.set_reference(_dev(rho))
    near = rho * (1.0 + 0.05 * rng.uniform(-1.0, 1.0, rho.shape))
    G, _ = mixed.residual(_dev(near))
    assert _rel(G.cpu().numpy(), st.G(near)) < 1e-6
    mixed.close()
