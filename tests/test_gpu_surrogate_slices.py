"""The judge over 16, 4 and 1 slices of the groups (few templates, more, the most; fewer than four groups): templates at
the ends of a large bank against the same ones in a small bank, and the small bank against the oracle.

A slice count changes only the order of the judge's FP64 sums of up to 12 groups: 12 eps of their magnitudes, 1e-14 on
1 - |sum| / sum; everything else is the same arithmetic."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2502_11823_amd import sft, synth
from parity_helpers import compare, gpu_scan, orc_scan

pytestmark = pytest.mark.gpu

HIDDEN, LAYERS = 16, 1


@pytest.mark.parametrize("n", [16384, 16385, 262144, 262145])
@pytest.mark.parametrize("n_sft", [1, 3, 4, 12])
def test_slices_agree(n_sft, n):
    w = synth.tiny(seed=1, n_templates=1, n_sft=n_sft, noise_series=False)
    ends = synth.uniform_bank(60, 1.19, 1.21, n_sft * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=n_sft)
    par = synth.mlp_init(13, HIDDEN, LAYERS)
    cfg = dict(mc_lo=1.19, mc_hi=1.21, q_lo=1.0, q_hi=2.0, lt_lo=float(np.log(600.0)), lt_hi=float(np.log(1400.0)),
               c_phi=0.05, c_amp=0.01, judge_tol=2.0, head=1)
    oracle.set_surrogate(par, cfg, HIDDEN, LAYERS)
    kw = dict(K=2, kernel="dirichlet", waveform="surrogate")
    mm = np.sort(orc_scan(w, ends, **kw)["mismatch"])
    cfg["judge_tol"] = 0.5 * (mm[29] + mm[30]) if mm[30] - mm[29] > 1e-12 else 1.0
    oracle.set_surrogate(par, cfg, HIDDEN, LAYERS)
    o = orc_scan(w, ends, **kw)
    s = sft.Surrogate(par, hidden=HIDDEN, layers=LAYERS, head=1, mc=(1.19, 1.21), q=(1.0, 2.0),
                      ln_tau=(cfg["lt_lo"], cfg["lt_hi"]), c_phi=0.05, c_amp=0.01, judge_tol=cfg["judge_tol"])
    data = sft.SFTData.from_workload(w, storage="f64")
    small = gpu_scan(data, ends, mismatch=True, precision="fp64", surrogate=s, **kw)
    compare(small, o, label="surrogate %d groups" % n_sft, tol_z=1e-9, tol_rho=1e-9, tol_hh=1e-9)
    idx = np.concatenate([np.arange(30), np.full(n - 60, 7), np.arange(30, 60)])
    big = gpu_scan(data, {k: v[idx] for k, v in ends.items()}, mismatch=True, precision="fp64", surrogate=s, **kw)
    s.close()
    for k in ("zp", "hhp", "rho", "flags", "n_used"):
        got = np.concatenate([big[k][:30], big[k][-30:]])
        assert np.allclose(got, small[k], rtol=1e-13, atol=1e-13 * np.abs(small[k]).max()), k
        assert np.all(big[k][30:-30] == big[k][30])
    got = np.concatenate([big["mismatch"][:30], big["mismatch"][-30:]])
    assert np.max(np.abs(got - small["mismatch"])) < 1e-14
