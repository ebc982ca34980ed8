"""The bf16 weight gradients (one product per problem over every (step, batch row),
operands staged contraction-major) against the oracle where their tiling can go
wrong: rows in all that do not fill a 32-row chunk, one row, steps of one row and of
31 and 33 (a chunk over many steps, and over two), widths that are not multiples of
8 (padded row pitches), of a row tile or of a column block, and both smaller tiles.
(The 256 x 256 tile runs in the full-batch parity case of the large-batch
workload.)  Rows of never-kept neurons are exact zeros."""
import dataclasses

import numpy as np
import pytest

import workloads
from tests._parity import TOL, compare, oracle_step, say, summary

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    dict(num_layers=1, num_dirs=1, input_dim=7, hidden=1, batch=1, seq_len=1),
    dict(num_layers=2, num_dirs=1, input_dim=9, hidden=129, batch=1, seq_len=70),
    dict(num_layers=2, num_dirs=2, input_dim=130, hidden=35, batch=31, seq_len=5, min_len=0),
    dict(num_layers=2, num_dirs=1, input_dim=65, hidden=64, batch=33, seq_len=3),
    dict(num_layers=2, num_dirs=1, input_dim=641, hidden=650, batch=3, seq_len=11),
    dict(num_layers=3, num_dirs=2, input_dim=40, hidden=96, batch=50, seq_len=2),
])
@pytest.mark.parametrize("mode", [(0.5, 0.5, 1), (0.7, 0.0, 0)])
def test_wgrad_rows_ragged(shape, mode):
    from oracle import masks as om
    from paper_2106_12089_amd.session import Session
    base = workloads.get_config("tiny")
    cfg = dataclasses.replace(base, name="wgrad_rows", dtype="bf16", loss="mse", **shape)
    wl = workloads.make_workload(cfg)
    p_nr, p_rh, compact = mode
    say(f"[gpu] wgrad rows {shape} p_nr={p_nr} p_rh={p_rh} compact={compact}")
    s = Session(wl, p_nr, p_rh, compact)
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    torch.cuda.synchronize()
    m_nr, m_rh = om.all_masks(cfg.mask_seed, 0, cfg.num_layers, cfg.num_dirs, cfg.seq_len, cfg.k_in, cfg.hidden,
                              p_nr, p_rh)
    gpu = s.outputs()
    errs = compare(gpu, oracle_step(wl, p_nr, p_rh, m_nr, m_rh))
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad
    for l in range(cfg.num_layers):
        for d in range(cfg.num_dirs):
            k = l * cfg.num_dirs + d
            assert np.all(gpu["dW"][k][~m_nr[l].any(axis=0)] == 0.0)
            assert np.all(gpu["dU"][k][~m_rh[l][d].any(axis=0)] == 0.0)
