"""The failure path of the persistent kernels, forced from the host: with a
zero barrier time-out every grid-barrier wait gives up at once, so every
workgroup leaves through the time-out path (no kernel spins or faults).  The
step must then report the failure through lstm_sd_status, write NaN into
every output it names, and a clean step on the same buffers afterwards must
match the oracle again.  Stacks in one launch (batch 20, 64), one bidirectional
layer, and the stress shape (batch 256, a launch per layer), whose clean step
after the failure is checked bit for bit against a fresh session's; and passes
of several launches of which one fails."""
import numpy as np
import pytest

import workloads
from tests._parity import TOL, compare, mode_rates, oracle_masks, oracle_step, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["lm_medium", "tagger", "seq2seq_enc"])
def test_forced_barrier_timeout_is_reported_then_recovers(name):
    from paper_2106_12089_amd import binding as B_
    from paper_2106_12089_amd.session import Session
    cfg = workloads.get_config(name)
    wl = workloads.make_workload(cfg)
    p = 0.5
    p_nr, p_rh, compact = mode_rates(cfg, "nrrh", p)
    s = Session(wl, p_nr, p_rh, compact)
    say(f"[gpu] forced barrier time-out {name}")
    B_.lstm_sd_set_barrier_timeout(0.0)
    try:
        s.masks(cfg.mask_seed, 0)
        s.forward()
        s.loss_grad()
        s.backward()
        with pytest.raises(B_.LstmSdError) as e:
            B_.lstm_sd_status(s.dims, s.workspace)
    finally:
        B_.lstm_sd_set_barrier_timeout(-1.0)
    assert e.value.code == B_.EHIP
    msg = str(e.value)
    assert "forward" in msg and "backward" in msg, msg
    out = s.outputs()
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        assert np.isnan(out[k]).all(), k
    for k in ("dW", "dU", "db"):
        for i, a in enumerate(out[k]):
            assert np.isnan(a).all(), (k, i)

    say(f"[gpu] clean step after the failure {name}")
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    B_.lstm_sd_status(s.dims, s.workspace)          # no error now
    torch.cuda.synchronize()
    gpu = s.outputs()
    m_nr, m_rh = oracle_masks(cfg, p_nr, p_rh)
    ref = oracle_step(wl, p_nr, p_rh, m_nr, m_rh)
    errs = compare(gpu, ref)
    say("   errs max", max(errs.values()))
    bad = {k: v for k, v in errs.items() if not v <= TOL[cfg.dtype]}
    assert not bad, bad


def test_forced_barrier_timeout_large_batch_recurrences():
    from paper_2106_12089_amd import binding as B_
    from paper_2106_12089_amd.session import Session
    cfg = workloads.get_config("stress")
    wl = workloads.make_workload(cfg)
    p_nr, p_rh, compact = mode_rates(cfg, "nrrh", 0.5)
    s = Session(wl, p_nr, p_rh, compact)
    say("[gpu] forced barrier time-out stress")
    B_.lstm_sd_set_barrier_timeout(0.0)
    try:
        s.masks(cfg.mask_seed, 0)
        s.forward()
        s.loss_grad()
        s.backward()
        with pytest.raises(B_.LstmSdError) as e:
            B_.lstm_sd_status(s.dims, s.workspace)
    finally:
        B_.lstm_sd_set_barrier_timeout(-1.0)
    assert e.value.code == B_.EHIP
    out = s.outputs()
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        assert np.isnan(out[k]).all(), k
    for k in ("dW", "dU", "db"):
        for i, a in enumerate(out[k]):
            assert np.isnan(a).all(), (k, i)

    say("[gpu] clean step after the failure stress")
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    B_.lstm_sd_status(s.dims, s.workspace)
    torch.cuda.synchronize()
    got = s.outputs()
    f = Session(wl, p_nr, p_rh, compact)
    f.masks(cfg.mask_seed, 0)
    f.forward()
    f.loss_grad()
    f.backward()
    torch.cuda.synchronize()
    ref = f.outputs()
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        assert np.array_equal(got[k], ref[k]), k
    for k in ("dW", "dU", "db"):
        for i, (a, b) in enumerate(zip(got[k], ref[k])):
            assert np.array_equal(a, b), (k, i)


@pytest.mark.parametrize("dtype,L,D,H,B", [
    ("bf16", 2, 2, 40, 20),           # a launch per layer
    ("f32", 2, 2, 40, 20),
    ("bf16", 1, 2, 520, 300),         # several launches of row groups
    ("bf16", 5, 1, 24, 17),           # more layers than one launch takes
    ("f32", 5, 1, 24, 17),
])
@pytest.mark.parametrize("which", [0, 1])
def test_one_launch_of_several_times_out(dtype, L, D, H, B, which, monkeypatch):
    """A barrier time-out in one persistent launch of a pass that takes several (a zero
    bound for that launch alone): what the launches before and after it wrote is poisoned
    all the same, and the next pass is clean."""
    import dataclasses
    from paper_2106_12089_amd import binding as B_
    from paper_2106_12089_amd.session import Session
    cfg = dataclasses.replace(workloads.get_config("tiny"), name="fail", dtype=dtype, loss="mse", num_layers=L,
                              num_dirs=D, input_dim=24, hidden=H, batch=B, seq_len=3)
    wl = workloads.make_workload(cfg)
    say(f"[gpu] one launch fails {dtype} L={L} D={D} H={H} B={B} which={which}")

    def step(s, fwd, bwd):
        s.masks(cfg.mask_seed, 0)
        monkeypatch.setenv("LSTM_SD_FAIL_LAUNCH", str(which) if fwd else "")
        s.forward()
        s.loss_grad()
        monkeypatch.setenv("LSTM_SD_FAIL_LAUNCH", str(which) if bwd else "")
        s.backward()
        torch.cuda.synchronize()
        monkeypatch.setenv("LSTM_SD_FAIL_LAUNCH", "")
        return s.outputs()

    ref = step(Session(wl, 0.5, 0.3, 1), False, False)
    s = Session(wl, 0.5, 0.3, 1)
    out = step(s, True, False)
    with pytest.raises(B_.LstmSdError, match="forward"):
        B_.lstm_sd_status(s.dims, s.workspace)
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        assert np.isnan(out[k]).all(), k
    out = step(s, False, True)
    with pytest.raises(B_.LstmSdError, match="backward"):
        B_.lstm_sd_status(s.dims, s.workspace)
    assert np.isfinite(out["y"]).all()
    for k in ("dx", "dh0", "dc0"):
        assert np.isnan(out[k]).all(), k
    # (fp32 writes a layer's weight gradients before the next layer's recurrence runs;
    # bf16 at these sizes writes all of them at the end)
    low = L * D if dtype == "bf16" else D
    for k in ("dW", "dU", "db"):
        for i, a in enumerate(out[k][:low]):
            assert np.isnan(a).all(), (k, i)
    out = step(s, False, False)
    B_.lstm_sd_status(s.dims, s.workspace)
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        assert np.array_equal(out[k], ref[k]), k
