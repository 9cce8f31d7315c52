"""The rows that pad a batch to a multiple of 16 have no part in the gradients, also where a row of zero inputs
overflows: a unit whose bias only the batch's own inputs cancel."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2502_11823_amd import synth

torch = pytest.importorskip("torch")
from paper_2502_11823_amd import sft  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,layers", [(16, 1), (16, 2), (48, 3), (128, 4)])
@pytest.mark.parametrize("B", [1, 15, 17, 100])
def test_overflow_in_the_padding(hidden, layers, B):
    par = synth.mlp_init(31 + hidden, hidden, layers).astype(np.float32)
    par[0], par[3 * hidden] = -3e37, 3e37               # unit 0: W[0][0] u_0 + b[0] = 0 at u_0 = 1
    par[hidden] = par[2 * hidden] = 0.0
    nxt = 4 * hidden                                     # its weights into the next layer: 3e37 x 100 overflows
    par[nxt:nxt + (hidden if layers > 1 else 2)] = 100.0
    g = np.random.default_rng(B)
    u = g.uniform(-1, 1, (B, 3)).astype(np.float32)
    u[:, 0] = 1.0
    y = g.normal(size=(B, 2)).astype(np.float32)
    s = sft.Surrogate(par, hidden=hidden, layers=layers)
    loss, grad = s.loss_grad(torch.as_tensor(u, device="cuda"), torch.as_tensor(y, device="cuda"))
    s.close()
    lo, go = omlp.loss_and_grad(par, u.astype(np.float64), y.astype(np.float64), hidden, layers)
    assert abs(float(loss.cpu()[0]) - lo) < 1e-6 * lo
    # the bound of the other tests of the step: 1e-5 of a block's norm
    off, grad = 0, grad.cpu().numpy().astype(np.float64)
    for ni, no in omlp.shapes(hidden, layers):
        for n in (ni * no, no):
            assert np.linalg.norm(grad[off:off + n] - go[off:off + n]) < 1e-5 * np.linalg.norm(go[off:off + n]), (ni, no, n)
            off += n
