"""Factorisation and solve of the coarse matrix at the edges of its forms: the
half band width kl is 3 b (diffusion) or 8 b + 1 (elasticity) for b boxes in x.
kl <= 48 runs in LDS, 49 .. 112 on eight wavefronts with its windows in global
memory, wider bands unblocked; row counts leave every kind of last panel.

Tolerance: two LU factorisations and two substitutions each of A0 and of the
local Jacobians, cond ~ 1e4 each, with the band's few hundred operations per
entry: 1e-10 of the largest entry."""
import numpy as np
import pytest

import synth
from oracle import NHProblem, P1Problem, Schwarz
from tests._lib import ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _check(case, P, u):
    from paper_2410_24138_amd import Solver
    S = Schwarz(P, "additive")
    s = Solver(case, coupling="additive")
    v = np.random.default_rng(9).normal(size=u.size)
    for a, ref in ((s.precond_residual(u), S.evaluate(u)), (s.tangent(v), S.tangent(v))):
        a = a.cpu().numpy()
        assert np.abs(a - ref).max() <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("boxes", [(15, 3), (16, 2), (17, 2), (21, 3), (37, 2), (38, 2)])
def test_diffusion(boxes):
    bx, by = boxes
    modes = synth.fourier_modes(3)
    case = synth.diffusion_case(3 * bx, 3 * by, synth.even_cuts(3 * bx, bx), synth.even_cuts(3 * by, by),
                                1, two_level=True, forcing=lambda p: synth.fourier_eval(p, modes))
    P = P1Problem(case)
    _check(case, P, 0.2 * np.random.default_rng(bx).normal(size=P.N))


@pytest.mark.parametrize("boxes", [(5, 4), (6, 2), (6, 5), (8, 8), (13, 2), (14, 2)])
def test_elasticity(boxes):
    bx, by = boxes
    case = synth.small_elasticity_case(nx=3 * bx, ny=3 * by, boxes=boxes, overlap=1,
                                       traction=(0.0, -0.5), two_level=True)
    P = NHProblem(case)
    h = 1.0 / (3 * max(bx, by))
    _check(case, P, 0.02 * h * np.random.default_rng(bx).normal(size=P.ndof) * ~P.is_dir)
