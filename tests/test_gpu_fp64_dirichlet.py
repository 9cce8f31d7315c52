"""The FP64 Dirichlet scan (bins in pairs from the edges inwards, its own sine, logarithm, roots) against the
oracle: the narrowest and the widest windows, one and several detectors, windows cut by the stored band, and
frequencies on the bins and half way between them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2502_11823_amd import sft, synth
from parity_helpers import compare, gpu_scan, orc_scan

pytestmark = pytest.mark.gpu

# FP64 throughout: the phases reach 1e6 rad, known to 1e6 x 2^-53 = 1.1e-10 rad by their argument alone
TIGHT = dict(tol_z=1e-9, tol_rho=1e-9, tol_hh=1e-9)


@pytest.mark.parametrize("waveform", ["newton", "pn35"])
@pytest.mark.parametrize("K", [0, 1, 3, 4, 17, 64])
def test_windows(K, waveform):
    w = synth.tiny(seed=1, n_templates=1, n_sft=24, noise_series=False)
    bank = synth.uniform_bank(70, 1.19, 1.21, 24 * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=w.n_sft)
    kw = dict(K=K, kernel="dirichlet", precision="fp64", waveform=waveform)
    compare(gpu_scan(sft.SFTData.from_workload(w, storage="f64"), bank, **kw), orc_scan(w, bank, **kw),
            label="fp64 K=%d %s" % (K, waveform), **TIGHT)


@pytest.mark.parametrize("K", [4, 9, 33])
def test_detectors_and_band_edges(K):
    w = synth.ground(seed=5, n_templates=130, n_slots=40, n_det=3, k_lo=60, k_hi=200, t_end_pad=400.0)
    kw = dict(K=K, kernel="dirichlet", precision="fp64", a_plus=1.0, a_cross=1.0)
    g = gpu_scan(sft.SFTData.from_workload(w, storage="f64"), w.bank, **kw)
    o = orc_scan(w, w.bank, **kw)
    assert np.any(o["flags"]) and np.array_equal(g["flags"], o["flags"])
    # the band cuts norm bins of flagged templates: their errors in units of the largest norm
    compare(g, o, label="fp64 ground K=%d" % K, noise_scale=(o["hhp"].max(), o["hhx"].max()), tol_z=1e-9, tol_rho=1e-8,
            tol_hh=1e-9)


@pytest.mark.parametrize("off", [0.0, 2.0 ** -40, -2.0 ** -40, 0.25, 0.4999999])
def test_frequencies_on_and_between_bins(off):
    """One SFT, coalescence times chosen so that f T at its midpoint is an integer plus off."""
    w = synth.tiny(seed=2, n_templates=1, n_sft=1, noise_series=False)
    mc = np.full(50, 1.2)
    M = mc * 4.925490947641267e-6
    kappa = 300.0 + np.arange(50) + off
    tau = 5.0 * M * (8.0 * np.pi * M * kappa / w.t_sft) ** (-8.0 / 3.0)
    bank = dict(mc=mc, t_c=w.t_start[0] + 0.5 * w.t_sft + tau, phi_c=np.zeros(50), q=np.ones(50),
                a_first=np.zeros(50, np.int32), a_last=np.zeros(50, np.int32))
    kw = dict(K=4, kernel="dirichlet", precision="fp64")
    g = gpu_scan(sft.SFTData.from_workload(w, storage="f64"), bank, **kw)
    o = orc_scan(w, bank, **kw)
    e = np.abs(g["zp"] - o["zp"]) / np.maximum(np.abs(o["zp"]), np.sqrt(o["hhp"]))
    assert np.array_equal(g["flags"], o["flags"]) and e.max() < 1e-9
