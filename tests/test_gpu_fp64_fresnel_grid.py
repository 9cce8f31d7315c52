"""Scans whose default is the persistent grid (a counter that every launch clears): the scan, the plan's
replays and the allocation-free entry agree to the last bit, and with the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2502_11823_amd import sft, synth
from parity_helpers import compare, orc_scan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waveform", ["newton", "pn35"])
@pytest.mark.parametrize("n", [1, 2, 300, 1025])
def test_entries_agree(n, waveform):
    w = synth.tiny(seed=4, n_templates=1, n_sft=30, noise_series=False)
    bank = synth.uniform_bank(n, 1.19, 1.21, 30 * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=w.n_sft)
    kw = dict(K=4, kernel="auto", precision="fp64", waveform=waveform)
    data = sft.SFTData.from_workload(w, storage="f64")
    bt, opts = sft.bank_to_device(bank), sft.make_opts(**kw)
    outs = [sft.template_bank_scan(data, bt, opts), sft.template_bank_scan_noalloc(data, bt, opts, sft.alloc_out(n))]
    plan = sft.Plan(data, bt, opts)
    for _ in range(3):
        torch.cuda.synchronize()
        for v in plan.out.values():
            v.zero_()
        plan.launch()
        outs.append({k: v.clone() for k, v in plan.out.items()})
    torch.cuda.synchronize()
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k], outs[0][k]), k
    plan.close()
    g = {k: v.cpu().numpy() for k, v in outs[0].items()}
    g["zp"], g["zx"] = g["zp"][:, 0] + 1j * g["zp"][:, 1], g["zx"][:, 0] + 1j * g["zx"][:, 1]
    g["flags"] = g["flags"].astype(np.uint32)
    compare(g, orc_scan(w, bank, **kw), label="fp64 fresnel n=%d %s" % (n, waveform), tol_z=1e-9, tol_rho=1e-9, tol_hh=1e-9)


@pytest.mark.parametrize("n", [2, 300])
@pytest.mark.parametrize("K", [23, 24, 50])
def test_wide_windows_of_single_rows(K, n):
    """3.5PN templates on single rows with FP32 sums: the persistent grid from K = 24 on, every entry and replay."""
    w = synth.tiny(seed=4, n_templates=1, n_sft=30, noise_series=False)
    bank = synth.uniform_bank(n, 1.19, 1.21, 30 * 64.0 + 600.0, 9, q_lo=1.0, q_hi=2.0, n_sft=w.n_sft)
    kw = dict(K=K, kernel="auto", precision="fp32_kahan", waveform="pn35")
    data = sft.SFTData.from_workload(w, storage="f32")
    bt, opts = sft.bank_to_device(bank), sft.make_opts(**kw)
    outs = [sft.template_bank_scan(data, bt, opts), sft.template_bank_scan_noalloc(data, bt, opts, sft.alloc_out(n))]
    plan = sft.Plan(data, bt, opts)
    for _ in range(3):
        torch.cuda.synchronize()
        for v in plan.out.values():
            v.zero_()
        plan.launch()
        outs.append({k: v.clone() for k, v in plan.out.items()})
    torch.cuda.synchronize()
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k], outs[0][k]), k
    plan.close()
    g = {k: v.cpu().numpy() for k, v in outs[0].items()}
    g["zp"], g["zx"] = g["zp"][:, 0] + 1j * g["zp"][:, 1], g["zx"][:, 0] + 1j * g["zx"][:, 1]
    g["flags"] = g["flags"].astype(np.uint32)
    compare(g, orc_scan(w, bank, **kw), label="wide windows K=%d n=%d" % (K, n))
