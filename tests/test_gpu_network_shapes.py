"""The BF16 inference kernel's workgroup shapes: row counts at the edges of their tiles and of the rule that
chooses the number of wavefronts, every width, against the FP64 inference of the same network."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _net(mode, hidden, layers):
    from paper_2502_11823_amd import sft, synth
    return sft.Surrogate(synth.mlp_init(3, hidden, layers), hidden=hidden, layers=layers, head=1, inference=mode,
                         mc=(1.19, 1.21), q=(1.0, 2.0), ln_tau=(6.0, 9.0), c_phi=1.0, c_amp=1.0)


# 4096 rows per wavefront of the chip: 4 / 8 / 12 wavefronts per workgroup at 1, 16385, 40000, 49152, 49153 rows
@pytest.mark.parametrize("hidden,layers", [(32, 1), (32, 3), (64, 2), (96, 3), (128, 2), (128, 4)])
@pytest.mark.parametrize("n", [1, 15, 64, 129, 16385, 40000, 49152, 49153])
def test_bf16_rows(hidden, layers, n):
    u = torch.empty((n, 3), dtype=torch.float64, device="cuda").uniform_(-1, 1, generator=torch.Generator("cuda").manual_seed(n))
    y0, d0 = _net("fp64", hidden, layers).infer(u)
    # operands of 16 (split) and 8 significant bits, errors of independent units adding through each layer
    for mode, eps in (("bf16x3", 2.0 ** -16), ("bf16", 2.0 ** -8)):
        y, d = _net(mode, hidden, layers).infer(u)
        for a, b in ((y, y0), (d, d0)):
            scale = float(b.abs().max())
            assert float((a - b).abs().max()) < 8 * layers * eps * scale, (mode, scale)
