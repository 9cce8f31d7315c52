"""Combination of the partial sums of the chunks (finalize kernel): one template, groups of 8 and
of 64 templates with ragged ends, fewer chunks than slices, as many, one more, and many.

All sums are FP64 and only their order differs, so results agree with the one-chunk scan (whose
single partial needs no combination) to n_groups * eps of the sum of the terms' magnitudes:
256 * 1.1e-16 * a factor 4 for z (its terms' magnitudes add up to at most ~sqrt(n_groups) / 4 times
the noise level sqrt(hh)), i.e. 1e-12 relative to max(|z|, sqrt(hh)) and to hh."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def handle():
    from paper_2502_11823_amd import sft, synth
    w = synth.tiny(seed=11, n_templates=130, n_sft=256, noise_series=False)
    return w, sft.SFTData.from_workload(w, storage="f64")


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 64, 65, 130])
@pytest.mark.parametrize("order", ["given", "track"])
def test_chunk_counts_agree(handle, n, order):
    from paper_2502_11823_amd import sft
    w, data = handle
    bank = sft.bank_to_device({k: v[:n] for k, v in w.bank.items()})
    opts = sft.make_opts(K=4, kernel="dirichlet", precision="fp64", a_plus=1.0, a_cross=0.5)
    sft.set_tuning(data, block=64, chunk_groups=256, order=order)
    ref = {k: v.cpu().numpy() for k, v in sft.template_bank_scan(data, bank, opts).items()}
    scale = np.maximum(np.abs(ref["zp"]).max(axis=1), np.sqrt(ref["hhp"]))
    # 2, 4, 31, 32, 33, 64, 256 chunks of the 256 groups (the last one short in some)
    for cg in (128, 64, 9, 8, 7, 4, 1):
        sft.set_tuning(data, block=64, chunk_groups=cg, order=order)
        got = {k: v.cpu().numpy() for k, v in sft.template_bank_scan(data, bank, opts).items()}
        for k in ("flags", "n_used"):
            assert np.array_equal(got[k], ref[k]), (cg, k)
        for k in ("zp", "zx"):
            assert np.max(np.abs(got[k] - ref[k]) / scale[:, None]) < 1e-12, (cg, k)
        for k in ("hhp", "rho"):
            assert np.max(np.abs(got[k] - ref[k]) / ref[k]) < 1e-12, (cg, k)


def test_large_bank_keeps_whole_rows(handle):
    """65537 templates (groups of 64 with many chunks) against the same templates in a small bank."""
    from paper_2502_11823_amd import sft
    w, data = handle
    opts = sft.make_opts(K=4, kernel="dirichlet", precision="fp64", a_plus=1.0, a_cross=0.5)
    sft.set_tuning(data, block=64, chunk_groups=4)
    small = {k: v for k, v in w.bank.items()}
    reps = 65537 // 130 + 1
    big = {k: np.tile(v, reps)[:65537] for k, v in small.items()}
    a = sft.template_bank_scan(data, sft.bank_to_device(small), opts)
    b = sft.template_bank_scan(data, sft.bank_to_device(big), opts)
    for k in ("zp", "hhp", "rho"):
        x, y = a[k].cpu().numpy(), b[k].cpu().numpy()
        s = np.abs(x).max()
        assert np.max(np.abs(y[:130] - x)) < 1e-12 * s and np.max(np.abs(y[-17:] - x[65520 % 130:][:17])) < 1e-12 * s, k
    assert np.array_equal(a["n_used"].cpu().numpy(), b["n_used"].cpu().numpy()[:130])
