"""The running median of the noise estimate: block widths at the edges of its three algorithms (32-bit keys two
and four per lane, rank counting), spectra whose values tie in the keys, and ranges that the keys cannot hold,
against the medians of the periodogram of the returned bins (NumPy, FP64)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _strain(kind, n, n_seg, rng):
    x = rng.standard_normal((2, n * n_seg))
    if kind == "impulse":        # a flat spectrum: every value of a block equal up to rounding
        x[:] = 0.0
        x[:, 3::n] = 1.0
    elif kind == "tones":        # a few values 1e13 above the rest, and every second bin far below
        t = np.arange(n * n_seg)
        x = 1e-3 * x + 1e4 * np.cos(2 * np.pi * 5 * t / n) + 1e4 * np.cos(2 * np.pi * (n // 4) * t / n)
    elif kind == "zeros":
        x[0, :n] = 0.0
        x[1, n:] *= 1e-150       # subnormal and zero periodogram values
    elif kind == "even":         # a period of n / 2: odd bins hold rounding noise only
        h = x[:, : n // 2]
        x = np.tile(h, (1, 2 * n_seg))
    return x


@pytest.mark.parametrize("kind", ["noise", "impulse", "tones", "zeros", "even"])
@pytest.mark.parametrize("n,w", [(64, 16), (128, 32), (256, 1), (256, 33), (512, 31), (512, 32), (512, 96), (512, 97),
                                 (1024, 50), (2048, 0), (4096, 25), (4096, 95), (8192, 64)])
def test_median_of_blocks(n, w, kind):
    from paper_2502_11823_amd import sft
    rng = np.random.default_rng(n + w)
    M, n_seg, dt = n // 2, 3, 1.0 / 128.0
    x = _strain(kind, n, n_seg, rng)
    bins, psd, keep = sft.make_sfts(torch.as_tensor(x, device="cuda"), n, dt, 0, M + 1, w)
    X = bins.cpu().numpy()
    X = X if np.iscomplexobj(X) else X[..., 0] + 1j * X[..., 1]
    X = X.reshape(2, n_seg, M + 1) / dt
    P = X.real ** 2 + X.imag ** 2
    s0 = np.clip(np.arange(M + 1) - w, 0, M - 2 * w)
    med = np.sort(P[..., s0[:, None] + np.arange(2 * w + 1)], -1)[..., w]
    B = sum(1.0 / (2 * w + 1 - i) for i in range(w + 1))
    ref = med * dt * dt * 2.0 / (n * dt * B)
    got = psd.cpu().numpy().reshape(2, n_seg, M + 1)
    assert (keep.cpu().numpy() == 1).all()
    # the bins are rounded by dt once more, the periodogram and the scale a few times: 16 ulp; dt^2 is exact
    # (a power of two), so subnormal values keep their spacing
    assert np.all(np.abs(got - ref) <= 16 * 2.0 ** -52 * ref + 1e-320)
