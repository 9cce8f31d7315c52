"""The training step (loss, gradients) at the edges of its kernels, against FP64 backpropagation."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2502_11823_amd import synth

torch = pytest.importorskip("torch")
from paper_2502_11823_amd import sft  # noqa: E402

pytestmark = pytest.mark.gpu


def blocks(hidden, layers):
    off, out = 0, []
    for i, (ni, no) in enumerate(omlp.shapes(hidden, layers)):
        out += [("W%d" % i, slice(off, off + ni * no)), ("b%d" % i, slice(off + ni * no, off + ni * no + no))]
        off += ni * no + no
    return out


@pytest.mark.parametrize("hidden,layers,B", [(16, 1, 1), (16, 2, 17), (32, 2, 15), (48, 3, 64), (80, 2, 65), (96, 4, 129),
                                             (112, 2, 1000), (128, 1, 4096), (128, 8, 130), (128, 4, 4097), (64, 3, 9000),
                                             (40, 2, 300), (144, 2, 100)])
def test_loss_grad_edges(hidden, layers, B):
    """Loss and gradient at the edges of the fused step (widths of 16 NT up to 128, one row, ragged row
    tiles and slices, one layer, eight) and of the layer-by-layer path (other widths) against FP64.

    Tolerance: each gradient element is an FP32 sum over the batch of products of FP32 chains
    (layers * hidden terms deep); rounding in quadrature gives a few eps * sqrt(hidden * layers), below
    1e-5 of the block's norm for these sizes."""
    par = synth.mlp_init(31 + hidden, hidden, layers)
    g = np.random.default_rng(B)
    u = g.uniform(-1, 1, (B, 3)).astype(np.float32)
    y = g.normal(size=(B, 2)).astype(np.float32)
    s = sft.Surrogate(par, hidden=hidden, layers=layers)
    loss, grad = s.loss_grad(torch.as_tensor(u, device="cuda"), torch.as_tensor(y, device="cuda"))
    lo, go = omlp.loss_and_grad(par, u.astype(np.float64), y.astype(np.float64), hidden, layers)
    assert abs(float(loss.cpu()[0]) - lo) < 1e-6 * lo
    grad = grad.cpu().numpy().astype(np.float64)
    for name, sl in blocks(hidden, layers):
        assert np.linalg.norm(grad[sl] - go[sl]) < 1e-5 * np.linalg.norm(go[sl]), name
    s.close()
