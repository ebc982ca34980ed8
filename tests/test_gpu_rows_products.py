"""The bf16 products over all (step, batch row) pairs -- the input product and the input
gradient -- against the oracle where their tiling can go wrong, through the vocabulary
head (any number of columns) and through layers of both directions: contractions that
fill no 32-column chunk or no step of two, row counts around a row tile, every tile
(64, 128 and 256 wide), sliced contractions, and large batches, where a layer takes them
or the products per step that skip the dropped neurons, by its rate, its width and how
full its tiles are.  The bound is that of the other bf16 parity tests."""
import dataclasses

import pytest

import workloads
from tests._parity import TOL, compare, oracle_step, say, summary
from tests.test_gpu_head import _check, _run_head, _synthetic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,F,V", [
    (1, 1, 3, 4),             # 64 x 64, one row
    (3, 43, 65, 132),         # 64 x 64, two row tiles and a row
    (5, 13, 31, 5004),        # gradient sliced over workgroups, output rows not a multiple of 4
    (2, 70, 132, 6148),       # the same, rows a multiple of 4, two row tiles
    (33, 32, 40, 4100),       # product 64 x 64, a short contraction
    (20, 32, 401, 4100),      # product 128 x 128
    (33, 64, 40, 4100),       # the same, a short contraction
    (9, 127, 1999, 516),      # gradient 64 x 64, 16 column tiles
    (11, 127, 1999, 516),     # gradient 128 x 128
    (16, 128, 40, 32768),     # product 256 x 256
    (26, 255, 2045, 68),      # gradient 256 x 256
])
@pytest.mark.parametrize("p,compact", [(0.5, 1), (0.3, 0)])
def test_head_products(T, B, F, V, p, compact):
    say(f"[gpu] rows products head T={T} B={B} F={F} V={V} p={p} compact={compact}")
    cfg, wl, y = _synthetic("rows", T, B, F, V, dtype="bf16", seed=F)
    got, ref, m = _run_head(cfg, wl, y, p, compact)
    _check(got, ref, TOL["bf16"])
    assert (got["dy"].transpose(0, 2, 1)[m == 0] == 0.0).all()


@pytest.mark.parametrize("shape,p_nr", [
    (dict(num_layers=2, num_dirs=2, input_dim=33, hidden=131, batch=21, seq_len=4), 0.5),
    (dict(num_layers=2, num_dirs=1, input_dim=140, hidden=70, batch=255, seq_len=2), 0.7),
    (dict(num_layers=2, num_dirs=1, input_dim=140, hidden=70, batch=256, seq_len=2), 0.7),
    (dict(num_layers=2, num_dirs=1, input_dim=140, hidden=70, batch=256, seq_len=2), 0.0),
    # per step over the kept neurons from 768 inputs on: products and gradients of one layer and of
    # both, at more and at half of them dropped; the last batch that fills its tiles and the first
    # that does not
    (dict(num_layers=2, num_dirs=1, input_dim=771, hidden=40, batch=218, seq_len=3), 0.7),
    (dict(num_layers=2, num_dirs=1, input_dim=1001, hidden=40, batch=256, seq_len=2), 0.5),
    (dict(num_layers=2, num_dirs=2, input_dim=61, hidden=390, batch=503, seq_len=2), 0.6),
    (dict(num_layers=1, num_dirs=1, input_dim=768, hidden=33, batch=217, seq_len=2), 0.7),
    (dict(num_layers=1, num_dirs=1, input_dim=768, hidden=33, batch=300, seq_len=2), 0.7),
    # (weights of a trained network's size: a larger recurrence multiplies every rounding over 64 steps)
    (dict(num_layers=1, num_dirs=1, input_dim=24, hidden=1030, batch=260, seq_len=64, weight_init="uniform",
          weight_scale=1030 ** -0.5), 0.5),
])
@pytest.mark.parametrize("compact", [1, 0])
def test_layer_products(shape, p_nr, compact):
    from oracle import masks as om
    from paper_2106_12089_amd.session import Session
    cfg = dataclasses.replace(workloads.get_config("tiny"), name="rows", dtype="bf16", loss="mse", **shape)
    wl = workloads.make_workload(cfg)
    say(f"[gpu] rows products {shape} p_nr={p_nr} compact={compact}")
    s = Session(wl, p_nr, 0.0, compact)
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    torch.cuda.synchronize()
    m_nr, m_rh = om.all_masks(cfg.mask_seed, 0, cfg.num_layers, cfg.num_dirs, cfg.seq_len, cfg.k_in, cfg.hidden,
                              p_nr, 0.0)
    errs = compare(s.outputs(), oracle_step(wl, p_nr, 0.0, m_nr, m_rh))
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad
