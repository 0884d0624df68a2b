"""The network's gradient at row counts next to its tiles (32-row and 64-row
tiles, splits of the batch by whole 64-row steps, at most 8 of them), against
the FP64 oracle.  bfloat16 operands (2^-9 relative, four layers of products
with independent roundings): 2e-2 of the gradient's 2-norm, layer by layer."""
import numpy as np
import pytest

import synth
from oracle import guess
from tests._lib import ensure_built

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 8, 31, 33, 64, 65, 511, 513, 577])
def test_gradient_rows(rows):
    ensure_built()
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_24138_amd import Solver
    s = Solver(synth.small_case(n=12, boxes=3, overlap=1))
    w = synth.mlp_init(3)
    X, T = synth.mlp_batch(rows, rows)
    s.guess_set_model(w)
    g, loss = s.guess_loss_grad(X, T)
    ref_loss, ref = guess.loss_grad(w.astype(np.float64), X.astype(np.float64), T.astype(np.float64))
    g = g.cpu().numpy().astype(np.float64)
    assert abs(loss - ref_loss) <= 2e-2 * ref_loss
    at = 0
    for i, o in zip(guess.DIMS[:-1], guess.DIMS[1:]):
        for n in (i * o, o):
            a, b = g[at:at + n], ref[at:at + n]
            assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b)
            at += n
