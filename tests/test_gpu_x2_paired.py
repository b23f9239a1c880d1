"""The x passes of large grids in the row lengths compiled in one launch shape, against the oracle: two waves per row
pair in the FMT pass (rows past 384 in FP32 only; FP64 keeps one wave per field there) and four waves a block in
the other two, with an odd number of rows and a ragged last block; and the n3-only pass of every compiled length.
FP64 fields and G to 1e-12 of each field's maximum, FP32-mixed G 5 % away from its reference to 1e-6, adjoint
weights to 1e-5 (the bars of the parity tests)."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from oracle import adjoint as oracle_adjoint
from oracle import picard, residual
from paper_0910_1531_amd import _abi
from paper_0910_1531_amd.solver import from_problem
from test_gpu_x2_forms import LENGTHS as TUNED
from test_gpu_x2_forms import WIDE_BLOCKS, _density, _dev, _problem, _rel

pytestmark = pytest.mark.gpu

LENGTHS = [8, 9, 12, 18, 27, 36, 54, 72, 81, 108, 144, 162, 216, 243, 288, 324, 432, 486, 512]
FOUR_WAVES = 2048   # the launcher's rule: at least so many waves of 256 // n_x (at least 1) row pairs, all species


def _grid(nx, least):
    """(nx, ny, nz) with an odd number of rows and at least `least` waves of row pairs."""
    pw = max(1, 256 // nx)
    rows = [(a, b) for a in (9, 27, 81, 243) for b in (27, 81, 243) if a <= b]
    ny, nz = next(r for r in sorted(rows, key=lambda r: r[0] * r[1]) if ((r[0] * r[1] + 1) // 2) // pw >= least)
    return (nx, ny, nz)


@pytest.mark.parametrize("nx", LENGTHS)
def test_large_grids(nx):
    p = _problem(_grid(nx, max(WIDE_BLOCKS + 1, -(-FOUR_WAVES // 3))), S=3)
    st = residual.Setup(p)
    rho = _density(p)
    ev = st.evaluate(rho)
    print(f"  {p.n}", file=sys.stderr, flush=True)
    sol = from_problem(p)
    out = sol.operators(_dev(rho))
    for key, ref in (("n", ev["n"]), ("dphi", ev["dphi"])):
        for k in range(10):
            assert _rel(out[key][k].cpu().numpy(), ref[k]) < 1e-12 or np.max(np.abs(ref[k])) < 1e-12, (key, k)
    del out
    G, r = sol.residual(_dev(rho))
    assert _rel(G.cpu().numpy(), ev["G"]) < 1e-12
    assert r == pytest.approx(st.residual_norm(st.sqnorm(rho - ev["G"])), rel=1e-12)
    # FP32-mixed against FP64 at a second density
    near = _dev(_density(p, 3, 0.05) * rho / np.where(rho > 0, p.initial_density(), 1.0))
    want, _ = sol.residual(near)
    mixed = from_problem(p, precision=_abi.DFT_FP32_MIXED)
    mixed.set_reference(_dev(rho))
    G, _ = mixed.residual(near)
    assert float((G - want).abs().max() / want.abs().max()) < 1e-6
    mixed.close()
    sol.close()


@pytest.mark.parametrize("functional", ["rosenfeld", "whitebear"])
@pytest.mark.parametrize("nx", [27, 54, 108, 162, 243, 288, 486])
def test_alternative_functionals(nx, functional):
    p = _problem(_grid(nx, WIDE_BLOCKS + 1), functional)
    st = residual.Setup(p)
    rho = _density(p)
    G_ref = st.G(rho)
    for prec, bar in ((_abi.DFT_FP64, 1e-12), (_abi.DFT_FP32_MIXED, 3e-6)):   # 15 % from the reference
        sol = from_problem(p, precision=prec)
        sol.set_reference(_dev(p.initial_density() * 0.5 + rho * 0.5))
        G, _ = sol.residual(_dev(rho))
        assert _rel(G.cpu().numpy(), G_ref) < bar
        sol.close()


@pytest.mark.parametrize("nx,functional", [(36, "rslt"), (81, "whitebear"), (162, "rslt"), (288, "rslt")])
def test_hessian_product(nx, functional):
    p = _problem(_grid(nx, WIDE_BLOCKS + 1), functional)
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


@pytest.mark.parametrize("nx", sorted(LENGTHS + TUNED))
def test_n3_only(nx):
    # a wall dense enough that a search is rejected and the next one's full step takes n3 alone
    p = W.hard_wall(n=(nx, 9, 27), h=(2.4 / nx, 0.2, 0.2), eta=0.38)
    ref = picard.PicardState(residual.Setup(p), p.initial_density())
    sol = from_problem(p)
    rho = _dev(p.initial_density())
    for _ in range(4):
        a_ref = ref.step()
        a, r = sol.picard_step(rho)
        assert a == pytest.approx(a_ref, rel=1e-6, abs=1e-12)
        assert r == pytest.approx(ref.r, rel=1e-6)
    assert ref.npartial > 0
    assert sol.stats()["n3_evals"] == ref.npartial
    sol.close()
