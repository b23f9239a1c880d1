"""The line search's evaluations one by one: which of them each search makes (alpha = 1 in full or for n3
alone, amax / 2, amax, the fitted step), their counts and the steps taken are the oracle's, through single
steps, runs and solves, and for the points of a batch that are at different evaluations at a time.  Walls
dense enough that the search rejects steps and its cap falls below 1 (n3 alone).  An evaluation agrees with
the oracle to 1e-12 and the fit of a step divides by second differences of f, at 1e-3 of f or more here:
steps to 1e-6."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import picard, residual
from paper_0910_1531_amd.solver import Batch, from_problem

pytestmark = pytest.mark.gpu

SEARCHES = 8


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("kind", ["steps", "run", "runs"])
@pytest.mark.parametrize("p", [W.hard_wall(n=(12, 9, 24), eta=0.3), W.hs_wall_nm(0.35, n=(384, 1, 1))],
                         ids=["12x9x24", "384x1x1"])
def test_evaluations_of_the_oracle(p, kind):
    ref = picard.PicardState(residual.Setup(p), p.initial_density())
    for _ in range(SEARCHES):
        ref.step()
    assert ref.npartial > 0 and ref.rejected > 0
    sol = from_problem(p)
    rho = _dev(p.initial_density())
    if kind == "steps":
        alpha = [sol.picard_step(rho)[0] for _ in range(SEARCHES)]
        assert np.allclose(alpha, [h["alpha"] for h in ref.history], rtol=1e-6, atol=0.0)
    else:
        for n in ((SEARCHES,) if kind == "run" else (1, 0, SEARCHES - 1)):
            sol.run(rho, n)
    s = sol.stats()
    assert (s["g_evals"], s["n3_evals"], s["rejected"], s["iterations"]) == \
        (ref.nevals, ref.npartial, ref.rejected, ref.iters)
    assert abs(s["residual"] - ref.r) <= 1e-6 * ref.r
    assert np.max(np.abs(rho.cpu().numpy() - ref.rho)) <= 1e-6 * np.max(ref.rho)
    sol.close()


def test_batch_points_at_different_evaluations():
    ps = [W.hard_wall(n=(12, 9, 24), eta=eta) for eta in (0.1, 0.3, 0.2, 0.35)]
    batch = Batch(ps)
    rhos = [_dev(p.initial_density()) for p in ps]
    its, rs, sts = batch.solve(rhos, 1e-8, 20)
    seen = set()
    for i, p in enumerate(ps):
        sol = from_problem(p)
        rho = _dev(p.initial_density())
        it, r, st = sol.solve(rho, 1e-8, 20, raise_on_fail=False)
        assert (it, r, st) == (its[i], rs[i], sts[i])
        assert torch.equal(rho, rhos[i])
        a, b = sol.stats(), batch.stats(i)
        assert all(a[k] == b[k] for k in ("g_evals", "n3_evals", "rejected"))
        seen.add(a["n3_evals"] > 0)
        sol.close()
    assert seen == {True, False}
