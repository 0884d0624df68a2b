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
