"""The surrogate judge with a diverged network (finite outputs of any size): the mismatch stays in [0, 1], every
template is flagged and takes the 3.5PN waveform."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2502_11823_amd import sft, synth
from parity_helpers import compare, gpu_scan, orc_scan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inference", ["fp64", "bf16x3"])
@pytest.mark.parametrize("scale", [1e14, 1e17, 1e18, 1e19, 1e20, 1e30])
def test_diverged_network_falls_back(scale, inference):
    w = synth.tiny(seed=1, n_templates=1, n_sft=60, noise_series=False)
    bank = synth.uniform_bank(37, 1.19, 1.21, 60 * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=w.n_sft)
    par = synth.mlp_init(13, 32, 2)
    par[-66:] *= scale                      # the output layer
    s = sft.Surrogate(par, hidden=32, layers=2, head=1, mc=(1.19, 1.21), q=(1.0, 2.0),
                      ln_tau=(float(np.log(600.0)), float(np.log(4500.0))), c_phi=2.0, c_amp=1e-35, judge_tol=0.5,
                      inference=inference)
    kw = dict(K=4, kernel="dirichlet")
    g = gpu_scan(sft.SFTData.from_workload(w, storage="f64"), bank, mismatch=True, precision="fp64",
                 waveform="surrogate", surrogate=s, **kw)
    s.close()
    # 1 - |sum w u| / sum w with |u| <= 1, in FP64
    assert np.all(g["mismatch"] >= -1e-12) and np.all(g["mismatch"] <= 1.0)
    o = orc_scan(w, bank, waveform="pn35", **kw)
    o["flags"] = o["flags"] | oracle.F_SURROGATE_FALLBACK
    compare(g, o, label="diverged %g %s" % (scale, inference), tol_z=1e-9, tol_rho=1e-9, tol_hh=1e-9)


@pytest.mark.parametrize("c_phi", [2.0, 1e20])
def test_diverged_network_accepted(c_phi):
    """A tolerance above 1 accepts every chirp: those far above every band are flagged for it and for their drift."""
    w = synth.tiny(seed=1, n_templates=1, n_sft=8, noise_series=False)
    bank = synth.uniform_bank(37, 1.19, 1.21, 8 * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=w.n_sft)
    par = synth.mlp_init(13, 32, 2)
    par[-66:] *= 1e30
    cfg = dict(mc_lo=1.19, mc_hi=1.21, q_lo=1.0, q_hi=2.0, lt_lo=float(np.log(600.0)), lt_hi=float(np.log(1200.0)),
               c_phi=c_phi, c_amp=1e-35, judge_tol=2.0, head=1)
    oracle.set_surrogate(par, cfg, 32, 2)
    s = sft.Surrogate(par, hidden=32, layers=2, head=1, mc=(1.19, 1.21), q=(1.0, 2.0), ln_tau=(cfg["lt_lo"], cfg["lt_hi"]),
                      c_phi=c_phi, c_amp=1e-35, judge_tol=2.0)
    kw = dict(K=4, kernel="dirichlet", waveform="surrogate", delta_max=1.0, surrogate=s)
    g = gpu_scan(sft.SFTData.from_workload(w, storage="f64"), bank, precision="fp64", **kw)
    s.close()
    o = orc_scan(w, bank, **kw)
    assert np.array_equal(g["flags"], o["flags"]) and np.array_equal(g["n_used"], o["n_used"])
    assert np.any(o["flags"] & oracle.F_OUT_OF_BAND) and np.any(o["flags"] & oracle.F_TAYLOR_INVALID)
