"""A bank of one template (timestamp groups over the lanes) against the same template twice in a bank of
two, which runs the general kernel with the same series bounds (both lanes hold the same template).

The sums over the groups run in the same chunks and the same order, with the same terms: z agrees to
1e-10 of the noise level sqrt(hh) or of |z| (FP64: 1e-12), the norm likewise, whatever the chunks."""
import threading

import numpy as np
import pytest

from paper_2502_11823_amd import synth

torch = pytest.importorskip("torch")
from paper_2502_11823_amd import sft  # noqa: E402

pytestmark = pytest.mark.gpu


def check(data, bank1, opts, tol):
    two = {k: np.concatenate([v, v]) for k, v in bank1.items()}
    a = {k: v.cpu().numpy() for k, v in sft.template_bank_scan(data, sft.bank_to_device(bank1), opts).items()}
    b = {k: v.cpu().numpy()[:1] for k, v in sft.template_bank_scan(data, sft.bank_to_device(two), opts).items()}
    assert a["flags"][0] == b["flags"][0] and a["n_used"][0] == b["n_used"][0]
    s = max(np.abs(b["zp"]).max(), np.abs(b["zx"]).max(), np.sqrt(b["hhp"][0]))
    for k in ("zp", "zx"):
        assert np.max(np.abs(a[k] - b[k])) <= tol * s, k
    for k in ("hhp", "hhx", "rho"):
        assert abs(a[k][0] - b[k][0]) <= tol * max(abs(b[k][0]), 1.0 if k == "rho" else 0.0), k
    arg = {k: float(bank1[k][0]) for k in ("mc", "t_c", "phi_c", "q")}
    r = sft.inner_product(data, opts=opts, a_first=int(bank1["a_first"][0]), a_last=int(bank1["a_last"][0]), **arg)
    assert r["flags"] == a["flags"][0] and r["zp"] == complex(*a["zp"][0]) and r["rho"] == a["rho"][0]
    assert r["hhp"] == a["hhp"][0] and r["zx"] == complex(*a["zx"][0])


@pytest.mark.parametrize("n_det,n_slots", [(1, 1), (1, 63), (2, 64), (3, 65), (3, 700)])
@pytest.mark.parametrize("K,kernel,waveform", [(0, "auto", "newton"), (3, "auto", "newton"), (8, "auto", "newton"),
                                               (8, "dirichlet", "newton"), (9, "auto", "pn35"), (8, "auto", "pn35"),
                                               (32, "auto", "newton"), (64, "fresnel", "newton")])
def test_ground_f32(n_det, n_slots, K, kernel, waveform):
    # a short pad: the last SFTs leave the band, and lie past coalescence for the second template
    w = synth.ground(seed=n_slots + K, n_templates=3, n_slots=n_slots, n_det=n_det, t_end_pad=60.0)
    data = sft.SFTData.from_workload(w, storage="f32")
    opts = sft.make_opts(K=K, kernel=kernel, waveform=waveform, a_plus=1.0, a_cross=0.7, delta_max=1.0)
    b = {k: v[:1].copy() for k, v in w.bank.items()}
    check(data, b, opts, 1e-10)
    for cg in (1, 3, 64, 65, 200):   # groups per chunk around a wavefront's 64
        sft.set_tuning(data, block=64, chunk_groups=cg)
        check(data, b, opts, 1e-10)
    b["t_c"][0] -= 200.0
    b["a_first"][0], b["a_last"][0] = w.n_sft // 3, max(w.n_sft // 3, w.n_sft - 2)
    check(data, b, opts, 1e-10)


@pytest.mark.parametrize("K,kernel,waveform", [(4, "dirichlet", "newton"), (5, "dirichlet", "pn35"), (4, "auto", "newton"),
                                               (6, "auto", "pn35")])
def test_tiny_f64(K, kernel, waveform):
    w = synth.tiny(seed=5, n_templates=1, n_sft=130, noise_series=False)
    data = sft.SFTData.from_workload(w, storage="f64")
    check(data, w.bank, sft.make_opts(K=K, kernel=kernel, waveform=waveform, precision="fp64"), 1e-12)


def test_calls_from_several_threads():
    """More calls in flight than the handle keeps blocks for."""
    w = synth.ground(seed=9, n_templates=8, n_slots=200, n_det=2)
    data = sft.SFTData.from_workload(w, storage="f32")
    opts = sft.make_opts(K=8, a_plus=1.0, a_cross=1.0)
    args = [dict(mc=float(w.bank["mc"][i]), t_c=float(w.bank["t_c"][i]), phi_c=0.3 * i) for i in range(8)]
    ref = [sft.inner_product(data, opts=opts, **a) for a in args]
    got = [[] for _ in args]

    def work(i):
        for _ in range(20):
            got[i].append(sft.inner_product(data, opts=opts, **args[i]))
    ts = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for i, r in enumerate(ref):
        assert len(got[i]) == 20 and all(g == r for g in got[i])
