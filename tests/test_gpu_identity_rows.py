"""Identity rows (Dirichlet dofs inside a patch) of mixed-precision handles: the
local linear systems multiply them by a power of two, which must not show."""
import numpy as np
import pytest

import synth
from oracle import P1Problem, Schwarz
from tests._lib import ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _solver(case, **kw):
    from paper_2410_24138_amd import Solver
    return Solver(case, coupling="one_level", **kw)


# The refinement's stopping rule is that of the unscaled system.  beta = 0, so
# that binary64 needs one Newton step; the iterate is 1 and misses the Dirichlet
# value 0, so that the residual is 1 in the identity rows and about 1e-3 (the
# load) in the others.  The first step's linear residual is at most 1e-10 of
# that in binary32 as well, below the asked 1e-8, and one step has to do; a bound
# taken from the rows scaled to kappa's size would be 1e-5 or 1e-4 of it.  (From
# kappa = 1e7 on the residual's own rounding, some 4 kappa eps per row, reaches
# 1e-8.)
@pytest.mark.parametrize("kappa", [1e5, 1e6])
def test_refinement_where_the_iterate_misses_dirichlet_values(kappa):
    case = synth.diffusion_case(24, 10, synth.even_cuts(24, 2), synth.even_cuts(10, 1), 1, beta=0.0)
    case["elem_coef"] = np.full(len(case["conn"]), kappa)
    S = Schwarz(P1Problem(case), "one_level", inner_rtol=1e-8)
    u = np.ones(S.P.N)
    ref = S.evaluate(u)
    assert [q["its"] for q in S.state["sols"]] == [1, 1]
    for precision in ("fp64", "fp32_ir"):
        s = _solver(case, precision=precision, inner_rtol=1e-8)
        F = s.precond_residual(u).cpu().numpy()
        assert list(s.inner_iterations()) == [1, 1]
        # both stop at a residual of 1e-8 of about sqrt(n); ||J^{-1}|| <= 1
        assert np.abs(F - ref).max() <= 1e-7


# Elements whose vertices are all Dirichlet: no other row sees their
# coefficient, however far it lies outside the range of binary32 (2^129 and
# 2^-148), so the results are those of coefficient 1 there.  The solves stop at
# the same Newton step; the rest is rounding, bounded by cond(J_ii) eps ~ 1e3 *
# 1e-16 per solve: 1e-11 for F_x and 1e-10 for the tangent.
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("kappa", [2.0 ** 129, 2.0 ** -148])
def test_coefficients_outside_binary32_between_dirichlet_nodes(kappa, precision):
    case = synth.diffusion_case(12, 8, synth.even_cuts(12, 2), synth.even_cuts(8, 1), 1)
    fixed = np.zeros(len(case["xy"]), bool)
    fixed[case["dirichlet"]] = True
    corner = fixed[case["conn"]].all(axis=1)
    assert corner.any()
    case["elem_coef"] = np.where(corner, kappa, 1.0)
    S = Schwarz(P1Problem(case), "one_level")
    rng = np.random.default_rng(4)
    u, v = rng.normal(size=S.P.N), rng.normal(size=S.P.N)
    s = _solver(case, precision=precision)
    for got, ref, tol in ((s.precond_residual(u), S.evaluate(u), 1e-11),
                          (s.tangent(v), S.tangent(v), 1e-10)):
        assert np.abs(got.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
