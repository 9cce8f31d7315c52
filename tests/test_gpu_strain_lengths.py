"""SFTs of segments whose length is no power of two (Bluestein's transform up to 8190 samples, the
defining sum above) against numpy's FFT.

Tolerance: the transform makes eight passes of small DFTs, three chirp or spectrum products and the
unfolding, each adding about eps of the signal's rms in quadrature: sqrt(16) * 2 * 1.1e-16 ~ 1e-15 of
the spectrum's rms; the largest of a few thousand bins stays within a factor 10 of that, 1e-14.  The
defining sum drifts with the length of its rotation (256 steps between anchors): 1e-12."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the smallest, lengths at the edges of the transform sizes 512, 576, ... 8192 (n - 1 <= L), M prime,
# the study's lengths, the longest, and two beyond
LENGTHS = [18, 22, 100, 510, 514, 576, 578, 640, 642, 768, 770, 1026, 1152, 1154, 1280, 1282, 1536, 1538, 2050, 2302,
           2306, 2560, 2562, 3070, 3074, 4094, 4098, 4138, 4240, 4608, 4610, 5120, 5122, 6144, 6146, 8178, 8190, 8194,
           9000]


@pytest.mark.parametrize("n", LENGTHS)
def test_bins_match_numpy(n):
    from paper_2502_11823_amd import sft
    n_det, n_seg, dt = 2, 5, 0.025
    rng = np.random.default_rng(n)
    # an odd series length: the second detector's segments start at an odd 8-byte word
    x = rng.standard_normal((n_det, n * n_seg + 1 + (n // 2) % 2 * 2))
    x[0, 2 * n + n // 3] = np.nan           # a gap
    x[1, 3 * n] = np.inf
    k_lo = 0 if n % 4 else n // 8
    n_bins = n // 2 + 1 - k_lo if n % 3 else max(1, n // 2 - k_lo - 3)
    xt = torch.as_tensor(x, device="cuda")
    bins, psd, keep = sft.make_sfts(xt, n, dt, k_lo, n_bins, 0, s_white=0.05)
    bins, psd, keep = bins.cpu().numpy(), psd.cpu().numpy(), keep.cpu().numpy()
    tol = 1e-14 if n <= 8190 else 1e-12
    for d in range(n_det):
        for a in range(n_seg):
            gap = (d, a) in ((0, 2), (1, 3))
            assert keep[d, a] == (0 if gap else 1)
            if gap:
                assert not bins[d, a].any() and not psd[d, a].any()
                continue
            ref = dt * np.fft.rfft(x[d, a * n:(a + 1) * n])
            rms = np.sqrt(np.mean(np.abs(ref) ** 2))
            assert np.max(np.abs(bins[d, a] - ref[k_lo:k_lo + n_bins])) < tol * rms
            assert np.all(psd[d, a] == 0.05)


def test_large_offset_and_pure_tone():
    """A tone on a bin of a 4240-sample segment: every other bin holds rounding only."""
    from paper_2502_11823_amd import sft
    n, dt, k = 4240, 0.025, 517
    j = np.arange(3 * n)
    x = np.cos(2 * np.pi * ((j * k) % n) / n)[None, :]
    bins, _, _ = sft.make_sfts(torch.as_tensor(x, device="cuda"), n, dt, 0, n // 2 + 1, 0, s_white=1.0)
    b = bins.cpu().numpy()[0] / dt
    assert np.max(np.abs(b[:, k] - n / 2)) < 1e-14 * n / 2 * 10
    b[:, k] = 0
    assert np.max(np.abs(b)) < 1e-14 * n / 2 * 10
