"""SFTs of short segments whose length is no power of two (the defining sum below 82 samples, the transform from there)
against the sum in long double.

Tolerance: a bin is a sum of n products whose twiddles carry two roundings each; with unit normal samples its error
has an rms below eps sqrt(n) x sqrt(n / 12) for the running sum and 2 eps sqrt(n) for the twiddles, under 6 eps of the
spectrum's rms sqrt(n) at n = 80 (sqrt(80 / 12) + 2 = 4.6), and the largest of 2e4 bins stays within a factor 5 of it:
30 eps = 3.4e-15."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [18, 20, 22, 24, 26, 34, 40, 48, 50, 62, 66, 72, 78, 80, 82, 84])
@pytest.mark.parametrize("k_lo,part", [(0, 1.0), (3, 0.4)])
def test_bins_match_the_defining_sum(n, k_lo, part):
    from paper_2502_11823_amd import sft
    rng = np.random.default_rng(n)
    n_det, n_seg, dt = 2, 200, 0.025
    n_bins = max(1, int(part * (n // 2 + 1 - k_lo)))
    x = rng.standard_normal((n_det, n_seg * n + 5))     # the second detector starts at an odd 8-byte word
    x[1, 7 * n + n - 1] = np.nan
    bins, psd, keep = sft.make_sfts(torch.as_tensor(x, device="cuda"), n, dt, k_lo, n_bins, 0, s_white=0.05)
    bins, psd, keep = bins.cpu().numpy(), psd.cpu().numpy(), keep.cpu().numpy()
    assert keep[1, 7] == 0 and keep.sum() == n_det * n_seg - 1 and not bins[1, 7].any() and not psd[1, 7].any()
    psd[1, 7] = 0.05
    assert np.all(psd == 0.05)
    seg = x[:, :n_seg * n].reshape(n_det, n_seg, n)
    seg[1, 7] = 0.0
    a = (np.outer(np.arange(n), k_lo + np.arange(n_bins)) % n).astype(np.longdouble)
    a *= -2 * np.longdouble("3.14159265358979323846264338327950288") / n
    re, im = seg.astype(np.longdouble) @ np.cos(a), seg.astype(np.longdouble) @ np.sin(a)
    e = np.hypot((bins.real / dt - re).astype(float), (bins.imag / dt - im).astype(float))
    assert e.max() < 30 * 2.0 ** -53 * np.sqrt(n) + 2.0 ** -52 * np.hypot(re, im).astype(float).max()
