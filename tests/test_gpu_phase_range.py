"""Phases of any size: a phi_c that is no angle (2^51 quarter turns and beyond) still gives terms of modulus one,
with the sine and cosine of the phase as FP64 holds it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2502_11823_amd import sft, synth
from parity_helpers import compare, gpu_scan, orc_scan

pytestmark = pytest.mark.gpu


def _case(phi_c, **kw):
    w = synth.tiny(seed=3, n_templates=1, n_sft=20, noise_series=False)
    bank = synth.uniform_bank(40, 1.19, 1.21, 20 * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=w.n_sft)
    bank["phi_c"] = np.full(40, phi_c)
    g = gpu_scan(sft.SFTData.from_workload(w, storage="f64" if kw["precision"] == "fp64" else "f32"), bank, **kw)
    return g, orc_scan(w, bank, **kw)


@pytest.mark.parametrize("kernel,K", [("dirichlet", 4), ("dirichlet", 8), ("auto", 8), ("auto", 13)])
@pytest.mark.parametrize("waveform", ["newton", "pn35"])
@pytest.mark.parametrize("phi_c", [1e15, 4e15, -4e15, 6.1e15, -8.7e15])
def test_fp32_sums(phi_c, waveform, kernel, K):
    # FP64 phases and FP32 sums: the bounds of the ordinary phases
    g, o = _case(phi_c, K=K, kernel=kernel, precision="fp32_kahan", waveform=waveform)
    compare(g, o, label="phi_c %g %s %s" % (phi_c, waveform, kernel))


@pytest.mark.parametrize("kernel,K", [("dirichlet", 4), ("dirichlet", 9), ("auto", 4), ("auto", 9)])
@pytest.mark.parametrize("waveform", ["newton", "pn35"])
@pytest.mark.parametrize("phi_c", [1e15, 1.2e15, -4e15, 6.1e15, 1.3e18, -1.3e18, 7e21])
def test_fp64_sums(phi_c, waveform, kernel, K):
    # the bounds of the ordinary phases; the reduction's second constant of 2 pi is good to 1e-32 a turn
    g, o = _case(phi_c, K=K, kernel=kernel, precision="fp64", waveform=waveform)
    compare(g, o, label="phi_c %g %s %s" % (phi_c, waveform, kernel), tol_z=1e-9, tol_rho=1e-9, tol_hh=1e-9)


@pytest.mark.parametrize("kernel", ["dirichlet", "auto"])
@pytest.mark.parametrize("phi_c", [1e35, -1e120, 1.7e308])
def test_fp64_terms_stay_bounded(phi_c, kernel):
    # no digit of such a phase is left, but every term keeps its modulus: z of noise alone stays near sqrt(<h, h>)
    kw = dict(K=4, kernel=kernel, precision="fp64")
    g, _ = _case(phi_c, **kw)
    z, _ = _case(0.0, **kw)
    assert np.all(np.isfinite(g["zp"])) and np.all(np.abs(g["zp"]) <= 10 * np.sqrt(g["hhp"]))
    assert np.allclose(g["hhp"], z["hhp"], rtol=1e-12, atol=0)
