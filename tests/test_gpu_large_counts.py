"""Counts past what one row of a grid holds (2^32 threads) and the largest banks' form of the finalize kernel: the ends
of a large call against a small one, bit for bit where the sums are the same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2502_11823_amd import sft, synth

pytestmark = pytest.mark.gpu


def _free(gib):
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip("needs %d GiB of free device memory" % gib)


def _ends(n, n_sft, chunk):
    """The first and the last 300 of n templates, in the bank of n and in one of 600."""
    w = synth.tiny(seed=11, n_templates=1, n_sft=n_sft, noise_series=False)
    data = sft.SFTData.from_workload(w, storage="f64")
    sft.set_tuning(data, block=256, chunk_groups=chunk)
    opts = sft.make_opts(K=1, kernel="dirichlet", precision="fp64")
    mc = torch.full((n,), 1.2, dtype=torch.float64, device="cuda")
    ends = torch.linspace(1.19, 1.21, 600, dtype=torch.float64, device="cuda")
    mc[:300], mc[-300:] = ends[:300], ends[300:]
    t_c = n_sft * 64.0 + 600.0
    big = sft.template_bank_scan(data, dict(mc=mc, t_c=torch.full_like(mc, t_c)), opts)
    small = sft.template_bank_scan(data, dict(mc=ends, t_c=torch.full_like(ends, t_c)), opts)
    torch.cuda.synchronize()
    out = {k: (torch.cat([v[:300], v[-300:]]).cpu().numpy(), small[k].cpu().numpy()) for k, v in big.items()}
    del big, mc
    torch.cuda.empty_cache()
    return out


@pytest.mark.parametrize("n,n_sft,chunk", [(65536, 3, 1), (65600, 9, 3), (1 << 22, 12, 2), ((1 << 22) + 1, 1, 1)])
def test_template_per_thread(n, n_sft, chunk):
    for k, (a, b) in _ends(n, n_sft, chunk).items():
        # at most 6 chunks, added in order or over slices: 6 eps of the noise level
        assert np.max(np.abs(a - b)) <= (0 if a.dtype.kind == "i" else 1e-14 * np.abs(b).max()), k


def test_bank_of_more_than_2_30_templates():
    _free(170)
    for k, (a, b) in _ends((1 << 30) + 77, 1, 1).items():
        assert np.array_equal(a, b), k


@pytest.mark.parametrize("inference", ["bf16", "bf16x3", "fp64"])
def test_inference_of_more_than_2_30_rows(inference):
    _free(80)
    n = (1 << 30) + 77
    net = sft.Surrogate(synth.mlp_init(13, 32, 1), hidden=32, layers=1, inference=inference)
    u = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    ends = torch.linspace(-1, 1, 1800, dtype=torch.float64, device="cuda").reshape(600, 3)
    u[:300], u[-300:] = ends[:300], ends[300:]
    big, small = net.infer(u), net.infer(ends)
    torch.cuda.synchronize()
    for a, b in zip(big, small):
        assert torch.equal(torch.cat([a[:300], a[-300:]]), b) and torch.equal(a[n // 2], a[300])
    net.close()
    del big, u, a
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n_det", [1, 2])
def test_segments_of_more_than_one_launch(n_det):
    """More than 2^21 segments, of a length that takes the convolution."""
    n, n_seg = 90, ((1 << 21) + 8) // n_det
    x = torch.zeros((n_det, n * n_seg), dtype=torch.float64, device="cuda")
    ends = (torch.linspace(-1, 1, n_det * 6 * n, dtype=torch.float64, device="cuda") ** 3).reshape(n_det, 6 * n)
    x[:, :3 * n], x[:, -3 * n:] = ends[:, :3 * n], ends[:, 3 * n:]
    big = sft.make_sfts(x, n, 0.025, 5, 3, 0, s_white=0.05)
    small = sft.make_sfts(ends, n, 0.025, 5, 3, 0, s_white=0.05)
    torch.cuda.synchronize()
    for a, b in zip(big, small):
        assert torch.equal(torch.cat([a[:, :3], a[:, -3:]], 1), b)
    assert int(big[2].sum()) == n_det * n_seg and not bool(big[0][:, 3:-3].any())
