"""Restarted GMRES with short cycles, cut in the middle of a cycle and at its
end: step by step and in captured blocks, against the oracle's.  Two outer
steps with GMRES stopped early; both forms run the same Krylov steps (classical
Gram-Schmidt with reorthogonalisation against the oracle's modified one), so the
iterates differ by the rounding of the local solves: 1e-10 relative."""
import numpy as np
import pytest

import synth
from oracle import NKS, P1Problem, Schwarz
from tests._lib import ensure_built

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart,maxit", [(1, 3), (2, 4), (3, 7), (7, 7), (9, 8)])
@pytest.mark.parametrize("form", ["steps", "graph", "nks"])
def test_short_cycles(form, restart, maxit):
    ensure_built()
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_24138_amd import Solver
    from paper_2410_24138_amd.nls import FLAG_GRAPH
    case = synth.small_case(n=20, boxes=4, overlap=1, two_level=True, forcing_seed=6)
    S = Schwarz(P1Problem(case), "additive")
    kw = dict(maxit=2, gmres_rtol=1e-6, gmres_restart=restart, gmres_maxit=maxit)
    ref, st = NKS(S).solve(**kw) if form == "nks" else S.solve(**kw)
    s = Solver(case, coupling="additive", outer_maxit=2, gmres_restart=restart, gmres_maxit=maxit,
               flags=FLAG_GRAPH if form == "graph" else 0)
    lib_solve = s.solve_nks if form == "nks" else s.solve
    u, got, _ = lib_solve()
    assert got["outer_its"] == st["outer"] and got["gmres_its"] == st["gmres"]
    assert np.linalg.norm(u.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
