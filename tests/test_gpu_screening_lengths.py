"""The screening operator where its passes change kernel: compiled z lengths (several radii a launch) beside x or y
lengths outside the compiled ones, the run-time-length z kernel, eight-column tiles (z 192 to 256), and the lengths
whose index arithmetic is redone (216, 243, 432, 486), with a last batch of fewer radii, against the oracle's
per-point dot product (1e-11 of the largest value, the bar of the other screening tests)."""
import math
import sys

import numpy as np
import pytest
import torch

import workloads as W
from oracle import screening
from paper_0910_1531_amd.solver import from_problem
from test_gpu_screening import _kmax

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


X_OUTSIDE = [((576, 1, 8), 2), ((6, 9, 27), 3), ((768, 1, 9), 1), ((4, 3, 243), 5)]
Y_OUTSIDE = [((16, 6, 18), 2), ((8, 4, 108), 3)]
Z_OUTSIDE = [((9, 8, 6), 3), ((8, 1, 576), 1)]
LONG = [((8, 2 if L < 300 else 1, L), 3 if L % 2 else 2) for L in (192, 216, 243, 256, 288, 384, 432, 486, 512)]


@pytest.mark.parametrize("n,S", X_OUTSIDE + Y_OUTSIDE + Z_OUTSIDE + LONG)
def test_matches_the_dot_product(n, S):
    R = 0.1 + 0.02 * np.arange(S)
    p = W.Problem(name=f"screening{n}", n=n, h=(0.1, 0.09, 0.11), radius=R, valence=np.zeros(S),
                  rho_bulk=np.full(S, 0.5))
    f = W.random_density(p, seed=3, amplitude=0.5)
    rsc = W.screening_radius(p, 0.12, 0.3, seed=2)
    M = int(math.ceil(_kmax(p) * (rsc.max() - rsc.min()))) + 8
    sol = from_problem(p)
    out = sol.rfd_reference(_dev(f), _dev(rsc), M).cpu().numpy()
    ref = screening.reference(f, rsc, p.n, p.h)
    err = np.abs(out - ref).max() / np.abs(ref).max()
    print(f"  n={n} S={S} M={M}: {err:.1e}", file=sys.stderr, flush=True)
    assert err < 1e-11
    sol.close()
