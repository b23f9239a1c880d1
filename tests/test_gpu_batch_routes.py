"""Batches whose points run other kernels together than alone: the x pass (at most 384 blocks: one wave per
field, else two waves per row pair) and the z passes (few blocks of four columns: one wave per transform) count
the blocks of all points of a launch.  Either kernel does the same arithmetic in the same order, so densities,
residuals and iteration counts of a point in a batch equal those of the point alone bit for bit."""
import sys

import numpy as np
import pytest
import torch

from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import Batch, from_problem
from test_gpu_parity import mixture

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _blocks(n):
    """Blocks of one point: the x pass with one wave per field, a z pass of four-column tiles."""
    pairs = (n[1] * n[2] + 1) // 2
    pw = max(1, 256 // n[0])
    return -(-pairs // pw), -(-(n[1] * (n[0] // 2 + 1)) // 4)


# grid, points, and the limits (x pass, Z1, Z2) that the batch passes and one point does not
CASES = [((48, 48, 48), 4, (384, 640, 1100)), ((64, 64, 64), 2, (None, 640, 640)), ((32, 32, 96), 3, (384, 384, 384)),
         ((24, 24, 162), 4, (384, 256, 256)), ((36, 36, 36), 7, (384, 640, 1100)), ((27, 27, 27), 10, (384, 640, None))]


@pytest.mark.parametrize("functional", ["rslt", "whitebear"])
@pytest.mark.parametrize("precision", [_abi.DFT_FP64, _abi.DFT_FP32_MIXED])
@pytest.mark.parametrize("n,count,limits", CASES)
def test_points_change_kernel(n, count, limits, precision, functional):
    bx, bz = _blocks(n)
    for b, limit in ((bx, limits[0]), (bz, limits[1]), (bz, limits[2])):
        assert limit is None or b <= limit < b * count
    pts = []
    for i in range(count):
        p = mixture(n, h=tuple(2.6 / m for m in n), S=2, es=True, seed=i)
        p.hs_functional = functional
        pts.append(p)
    b = Batch(pts, precision=precision)
    rhos = [_dev(p.initial_density()) for p in pts]
    its, norms, sts = b.solve(rhos, 1e-8, 60)
    print(f"  {count} x {n} {functional} precision {precision}: iterations {its}, statuses {sts}", file=sys.stderr, flush=True)
    for i, p in enumerate(pts):
        sol = from_problem(p, precision=precision)
        x = _dev(p.initial_density())
        it, r, st = sol.solve(x, 1e-8, 60, raise_on_fail=False)
        # (a point that is not done by then stops at the same iterate; its residual may come from an FP32 evaluation
        # in the one and an FP64 evaluation in the other)
        assert (st, it) == (sts[i], its[i]) and (st != 0 or r == norms[i]), i
        assert torch.equal(x, rhos[i]), i
        sol.close()
    b.close()
