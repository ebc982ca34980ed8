"""Whole bf16 steps of large and ragged batches against the oracle: hidden sizes that are
not multiples of the 32-neuron chunk or of the 16-unit tile, batches that are not
multiples of a row group or of the 16-row MFMA tile, more row groups than one launch
takes, 256 rows and more, both directions, per-row lengths, and both modes; with the recurrences persistent and
with the per-step kernels, which run where a recurrence does not fit the device; and the
same bits from every repeat."""
import dataclasses

import numpy as np
import pytest

import workloads
from tests._parity import TOL, compare, oracle_step, say, summary

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(cfg, wl, p_nr, p_rh, compact):
    from oracle import masks as om
    from paper_2106_12089_amd.session import Session
    s = Session(wl, p_nr, p_rh, compact)
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    torch.cuda.synchronize()
    m_nr, m_rh = om.all_masks(cfg.mask_seed, 0, cfg.num_layers, cfg.num_dirs, cfg.seq_len, cfg.k_in,
                              cfg.hidden, p_nr, p_rh)
    return s.outputs(), oracle_step(wl, p_nr, p_rh, m_nr, m_rh)


@pytest.mark.parametrize("shape", [
    dict(num_layers=2, num_dirs=1, input_dim=70, hidden=45, batch=70, seq_len=5),
    dict(num_layers=1, num_dirs=2, input_dim=129, hidden=100, batch=19, seq_len=4),
    dict(num_layers=2, num_dirs=1, input_dim=64, hidden=1000, batch=130, seq_len=3),
    dict(num_layers=1, num_dirs=1, input_dim=33, hidden=512, batch=64, seq_len=6, min_len=0),
    dict(num_layers=2, num_dirs=2, input_dim=200, hidden=72, batch=300, seq_len=3),
    dict(num_layers=1, num_dirs=2, input_dim=48, hidden=40, batch=1030, seq_len=3),
])
@pytest.mark.parametrize("mode", [(0.5, 0.5, 1), (0.5, 0.5, 0), (0.3, 0.0, 1)])
def test_big_ragged(shape, mode):
    base = workloads.get_config("tiny")
    cfg = dataclasses.replace(base, name="big", dtype="bf16", loss="mse", **shape)
    wl = workloads.make_workload(cfg)
    p_nr, p_rh, compact = mode
    say(f"[gpu] big {shape} p_nr={p_nr} p_rh={p_rh} compact={compact}")
    gpu, ref = _run(cfg, wl, p_nr, p_rh, compact)
    errs = compare(gpu, ref)
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad
    if cfg.min_len is not None:
        valid = np.arange(cfg.seq_len)[:, None] < wl.lengths[None, :]
        assert np.all(gpu["y"][~valid] == 0.0)


@pytest.mark.parametrize("shape", [
    dict(num_layers=2, num_dirs=1, input_dim=70, hidden=45, batch=70, seq_len=5),
    dict(num_layers=2, num_dirs=2, input_dim=200, hidden=72, batch=300, seq_len=3),
])
@pytest.mark.parametrize("mode", [(0.5, 0.5, 1), (0.5, 0.5, 0)])
def test_big_per_step_kernels(shape, mode, monkeypatch):
    """The recurrences as one launch per step (LSTM_SD_PERSIST=0)."""
    monkeypatch.setenv("LSTM_SD_PERSIST", "0")
    base = workloads.get_config("tiny")
    cfg = dataclasses.replace(base, name="big", dtype="bf16", loss="mse", **shape)
    wl = workloads.make_workload(cfg)
    p_nr, p_rh, compact = mode
    say(f"[gpu] big per step {shape} p_nr={p_nr} p_rh={p_rh} compact={compact}")
    gpu, ref = _run(cfg, wl, p_nr, p_rh, compact)
    errs = compare(gpu, ref)
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad


@pytest.mark.parametrize("mode", [(0.3, 0.0, 1), (0.5, 0.5, 1), (0.5, 0.5, 0)])
def test_big_repeats_bit_identical(mode):
    """The same step on the same masks gives the same bits every time: the
    exchanges of the recurrences and the products' accumulation orders leave
    no room for a race."""
    from paper_2106_12089_amd.session import Session
    base = workloads.get_config("tiny")
    cfg = dataclasses.replace(base, name="big", dtype="bf16", loss="mse", num_layers=2, num_dirs=1, input_dim=70,
                              hidden=45, batch=70, seq_len=5)
    wl = workloads.make_workload(cfg)
    p_nr, p_rh, compact = mode
    say(f"[gpu] big repeats p_nr={p_nr} p_rh={p_rh} compact={compact}")
    ref = None
    for it in range(6):
        s = Session(wl, p_nr, p_rh, compact)
        s.masks(cfg.mask_seed, 0)
        s.forward()
        s.loss_grad()
        s.backward()
        torch.cuda.synchronize()
        o = s.outputs()
        cur = {k: np.concatenate([np.ravel(a) for a in v]) if isinstance(v, list) else np.ravel(v)
               for k, v in o.items() if v is not None and k != "loss"}
        if ref is None:
            ref = cur
            continue
        diff = [k for k in ref if not np.array_equal(ref[k], cur[k])]
        assert not diff, (it, diff)
