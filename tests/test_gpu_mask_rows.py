"""The masked copies of x and h0 (bf16) against the oracle, through the whole step, at
every alignment of a row (widths that are a multiple of 8, 4, 2 and 1, below one piece of
8 columns, and the largest), with several rows to a workgroup's pass and one, and with an
input whose first element is not 16-byte aligned.  The bound is that of the other bf16
parity tests."""
import dataclasses

import pytest

import workloads
from tests._parity import TOL, compare, oracle_step, say, summary

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I,H,D,B,T,offset", [
    (1, 8, 1, 1, 1, 0),
    (7, 12, 2, 3, 5, 0),
    (64, 66, 2, 5, 9, 0),
    (20, 67, 1, 33, 4, 0),
    (64, 72, 2, 5, 4, 1),
    (64, 72, 1, 5, 4, 2),
    (2048, 40, 1, 3, 3, 0),
    (2045, 44, 1, 3, 3, 4),
    (2000, 24, 1, 61, 18, 0),     # four rows a thread, whole groups of eight mask bytes
    (1501, 21, 1, 61, 24, 0),     # four rows a thread, single mask bytes
])
def test_masked_copies(I, H, D, B, T, offset):
    from oracle import masks as om
    from paper_2106_12089_amd.session import Session
    cfg = dataclasses.replace(workloads.get_config("tiny"), name="copies", dtype="bf16", loss="mse", num_layers=2,
                              num_dirs=D, input_dim=I, hidden=H, batch=B, seq_len=T)
    wl = workloads.make_workload(cfg)
    say(f"[gpu] masked copies I={I} H={H} D={D} B={B} T={T} offset={offset}")
    s = Session(wl, 0.4, 0.3, 1)
    if offset:
        buf = torch.empty(s.x.numel() + offset, dtype=s.x.dtype, device=s.x.device)
        buf[offset:] = s.x.reshape(-1)
        s.x = buf[offset:].view(s.x.shape)
    s.masks(cfg.mask_seed, 0)
    s.forward()
    s.loss_grad()
    s.backward()
    torch.cuda.synchronize()
    m_nr, m_rh = om.all_masks(cfg.mask_seed, 0, 2, D, T, cfg.k_in, H, 0.4, 0.3)
    errs = compare(s.outputs(), oracle_step(wl, 0.4, 0.3, m_nr, m_rh))
    say("   errs", summary(errs))
    bad = {k: v for k, v in errs.items() if not v <= TOL["bf16"]}
    assert not bad, bad
