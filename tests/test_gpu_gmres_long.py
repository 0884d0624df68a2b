"""A GMRES cycle of more than 2,048 steps, whose totals per step go through global
memory (from 8,192 on they would exceed the LDS of a launch)."""
import numpy as np
import pytest

import synth
from oracle import P1Problem, Schwarz
from tests._lib import ensure_built

pytestmark = pytest.mark.gpu


# A linear problem (beta = 0), one outer step, and a negative tolerance, which
# nothing meets: the cycle runs through all its steps, most of them in directions
# that the solution does not need.  The step is the solution, to
# the rounding of the tangent (cond of DF_x below 1e4): 1e-10 relative.
def test_long_cycle():
    ensure_built()
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_24138_amd import Solver
    steps = 2100
    case = synth.diffusion_case(96, 92, synth.even_cuts(96, 3), synth.even_cuts(92, 3), 1, beta=0.0)
    P = P1Problem(case)
    s = Solver(case, coupling="one_level", outer_maxit=1, outer_rtol=1e-30, gmres_rtol=-1.0,
               gmres_restart=steps, gmres_maxit=steps)
    u, st, rc = s.solve()
    assert st["gmres_its"] == [steps]
    ref, st_ref = Schwarz(P, "one_level").solve(maxit=1, rtol=1e-30, gmres_rtol=1e-12,
                                                gmres_restart=300)
    assert np.linalg.norm(u.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
