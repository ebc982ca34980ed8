"""Vocabulary heads (bf16) whose gradient of the logits takes more than 32 bits of
bytes -- a step's block above 2 GiB, and a batch of one with two million columns, whose
32-row chunks span as many steps -- against the oracle, with only the rows that lie past
those bytes counting (every other target is ignored, so their gradients are zero).  The
bound is that of the other bf16 parity tests."""
import types

import numpy as np
import pytest

from oracle import head
from tests._parity import TOL, say
from tests.test_gpu_head import _check, _head

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,F,V,first", [
    (1, 32768, 8, 32800, 32740),      # a block of 2 GiB and two row tiles
    (2, 32768, 264, 32800, 65500),    # the same with the 256 x 256 tile
    (40, 1, 5, 2300004, 29),          # a chunk's rows 2 GiB apart
    (67, 1, 3, 2300004, 62),
])
def test_rows_past_two_gib(T, B, F, V, first):
    import workloads
    say(f"[gpu] large vocabulary T={T} B={B} F={F} V={V}")
    rng = np.random.default_rng(V)
    q = workloads.round_to_bf16
    cfg = types.SimpleNamespace(name="vocab", dtype="bf16", num_layers=1, seq_len=T, mask_seed=5)
    targets = np.full((T, B), -1, np.int32)
    targets.reshape(-1)[first:] = rng.integers(0, V, size=T * B - first)
    wl = types.SimpleNamespace(
        cfg=cfg, x=np.zeros((T, B, 1), np.float32), lengths=None,
        W_fc=q(rng.uniform(-0.3, 0.3, size=(F, V)).astype(np.float32)),
        b_fc=rng.uniform(-0.1, 0.1, size=(V,)).astype(np.float32), targets=targets)
    y = q(rng.normal(0.0, 1.0, size=(T, B, F)).astype(np.float32))
    h = _head(wl, 0.0, 1, cfg.mask_seed)
    h.forward(torch.from_numpy(y).cuda())
    h.backward()
    torch.cuda.synchronize()
    rows = np.arange(first, T * B)
    m = np.ones((len(rows), F), np.uint8)
    pick = lambda a: a.reshape(T * B, 1, -1)[rows]
    ref = head.head_step(pick(y), wl.W_fc, wl.b_fc, m, 0.0, pick(targets)[:, :, 0], None)
    at = torch.from_numpy(rows).cuda()
    dev = lambda t: t.reshape(T * B, 1, -1)[at].double().cpu().numpy()
    got = dict(z=dev(h.logits), dy=dev(h.dy), loss=float(h.loss.item()), dW=h.dW.double().cpu().numpy(),
               dc=h.db.double().cpu().numpy())
    _check(got, ref, TOL["bf16"])
    h.dy.view(T * B, F)[at] = 0.0
    assert not h.dy.any()                  # rows that do not count
