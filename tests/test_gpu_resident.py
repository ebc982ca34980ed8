"""The bf16 recurrences with register-resident weights against the oracle at the
edges of their tilings: hidden sizes around the 32-neuron chunk, the unit tiles
and the eight-chunk rounds of the waves (one unit, odd, 1537 and 2047), row
groups of 4 to 32 rows that do not divide the batch, more row groups than one
launch takes, stacks of up to four layers with their workers, both directions,
and lengths of zero.  The bound is that of the other bf16 parity tests."""
import dataclasses

import numpy as np
import pytest

import workloads
from tests._parity import TOL, compare, oracle_step, say, summary

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    dict(num_layers=1, num_dirs=1, input_dim=5, hidden=1, batch=1, seq_len=3),
    dict(num_layers=2, num_dirs=1, input_dim=9, hidden=33, batch=17, seq_len=4, min_len=0),
    dict(num_layers=4, num_dirs=1, input_dim=40, hidden=255, batch=20, seq_len=5),
    dict(num_layers=2, num_dirs=2, input_dim=31, hidden=257, batch=49, seq_len=3, min_len=0),
    dict(num_layers=3, num_dirs=1, input_dim=64, hidden=706, batch=5, seq_len=4),
    dict(num_layers=2, num_dirs=1, input_dim=16, hidden=1025, batch=33, seq_len=3),
    dict(num_layers=1, num_dirs=1, input_dim=16, hidden=1537, batch=18, seq_len=3),
    dict(num_layers=1, num_dirs=1, input_dim=16, hidden=2047, batch=3, seq_len=3),
    dict(num_layers=1, num_dirs=2, input_dim=24, hidden=520, batch=300, seq_len=3, min_len=0),
])
@pytest.mark.parametrize("mode", [(0.5, 0.5, 1), (0.3, 0.0, 0)])
def test_resident_recurrences_ragged(shape, mode):
    from oracle import masks as om
    from paper_2106_12089_amd.session import Session
    base = workloads.get_config("tiny")
    cfg = dataclasses.replace(base, name="resident", dtype="bf16", loss="mse", **shape)
    wl = workloads.make_workload(cfg)
    p_nr, p_rh, compact = mode
    say(f"[gpu] resident {shape} p_nr={p_nr} p_rh={p_rh} compact={compact}")
    s = Session(wl, p_nr, p_rh, compact)
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    torch.cuda.synchronize()
    m_nr, m_rh = om.all_masks(cfg.mask_seed, 0, cfg.num_layers, cfg.num_dirs, cfg.seq_len, cfg.k_in, cfg.hidden,
                              p_nr, p_rh)
    errs = compare(s.outputs(), oracle_step(wl, p_nr, p_rh, m_nr, m_rh))
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad
    if cfg.min_len is not None:
        valid = np.arange(cfg.seq_len)[:, None] < wl.lengths[None, :]
        assert np.all(s.outputs()["y"][~valid] == 0.0)
