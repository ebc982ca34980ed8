"""Inf and NaN in weight rows of neurons that are dropped at every step (bf16): the method
does not read those rows, so nothing of them may reach an output, on every path of the
forward products -- stacks with their product workers, layers one by one, row groups of a
large batch, products that skip the dropped neurons and products that multiply their
zeros, the per-step kernels, and the vocabulary head.  The reference is the oracle with
those rows zero; the bound is that of the other bf16 parity tests.  Rows of kept neurons
do reach the outputs."""
import dataclasses

import numpy as np
import pytest

import workloads
from tests._parity import TOL, compare, oracle_step, say, summary
from tests.test_gpu_head import _check, _head, _out_mask, _synthetic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
BAD = [float("inf"), float("nan"), float("-inf")]


def _spoil(host, dev, never):
    """Rows `never`: zeros in the reference's weights, Inf and NaN in the device's."""
    host[never] = 0.0
    rows = np.nonzero(never)[0]
    for i, k in enumerate(rows):
        dev[int(k)] = BAD[i % 3]
    return len(rows)


@pytest.mark.parametrize("shape,p_nr,persist", [
    (dict(num_layers=3, num_dirs=1, input_dim=60, hidden=45, batch=20, seq_len=3), 0.5, "1"),
    (dict(num_layers=2, num_dirs=2, input_dim=33, hidden=70, batch=37, seq_len=3), 0.5, "1"),
    (dict(num_layers=2, num_dirs=1, input_dim=780, hidden=70, batch=256, seq_len=3), 0.7, "1"),
    (dict(num_layers=1, num_dirs=1, input_dim=130, hidden=520, batch=300, seq_len=3), 0.3, "1"),
    (dict(num_layers=2, num_dirs=1, input_dim=60, hidden=45, batch=20, seq_len=3), 0.5, "0"),
])
def test_dropped_rows_are_not_read(shape, p_nr, persist, monkeypatch):
    from oracle import masks as om
    from paper_2106_12089_amd.session import Session
    monkeypatch.setenv("LSTM_SD_PERSIST", persist)
    cfg = dataclasses.replace(workloads.get_config("tiny"), name="nonfinite", dtype="bf16", loss="mse", **shape)
    wl = workloads.make_workload(cfg)
    say(f"[gpu] non-finite dropped rows {shape} p_nr={p_nr} persist={persist}")
    s = Session(wl, p_nr, 0.5, 1)
    m_nr, m_rh = om.all_masks(cfg.mask_seed, 0, cfg.num_layers, cfg.num_dirs, cfg.seq_len, cfg.k_in, cfg.hidden,
                              p_nr, 0.5)
    n = 0
    for l in range(cfg.num_layers):
        for d in range(cfg.num_dirs):
            k = l * cfg.num_dirs + d
            n += _spoil(wl.W[k], s.W[k], ~m_nr[l].any(axis=0))
            n += _spoil(wl.U[k], s.U[k], ~m_rh[l][d].any(axis=0))
    assert n >= 3 * cfg.num_layers
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    torch.cuda.synchronize()
    errs = compare(s.outputs(), oracle_step(wl, p_nr, 0.5, m_nr, m_rh))
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad


@pytest.mark.parametrize("T,B,F,V", [(2, 3, 50, 36), (3, 100, 40, 32768), (3, 40, 65, 6148)])
def test_dropped_rows_of_the_head_are_not_read(T, B, F, V):
    from oracle import head
    say(f"[gpu] non-finite dropped rows head T={T} B={B} F={F} V={V}")
    cfg, wl, y = _synthetic("nonfinite", T, B, F, V, dtype="bf16", seed=F)
    h = _head(wl, 0.5, 1, cfg.mask_seed)
    m = _out_mask(cfg, F, 0.5)
    assert _spoil(wl.W_fc, h.W_fc, ~m.astype(bool).any(axis=0)) >= 3
    h.forward(torch.from_numpy(y).cuda())
    h.backward()
    torch.cuda.synchronize()
    _check(h.outputs(), head.head_step(y, wl.W_fc, wl.b_fc, m, 0.5, wl.targets, wl.lengths), TOL["bf16"])


def test_kept_rows_reach_the_outputs():
    """NaN in one kept row: its gate's sums, and with them every output of the unit, are NaN."""
    from paper_2106_12089_amd.session import Session
    cfg = dataclasses.replace(workloads.get_config("tiny"), name="nonfinite", dtype="bf16", loss="mse", num_layers=1,
                              num_dirs=1, input_dim=40, hidden=45, batch=20, seq_len=3)
    wl = workloads.make_workload(cfg)
    say("[gpu] non-finite kept rows")
    for which in ("W", "U"):
        s = Session(wl, 0.0, 0.0, 1)
        getattr(s, which)[0][7, 45 + 3] = float("nan")          # the forget gate of unit 3
        s.masks(cfg.mask_seed, 0)
        s.forward()
        torch.cuda.synchronize()
        y = s.outputs()["y"]
        assert np.isnan(y[:, :, 3]).all() and np.isfinite(np.delete(y[0], 3, axis=1)).all(), which
