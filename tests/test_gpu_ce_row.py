"""The one-pass loss and gradient of bf16 heads against the oracle where its split can go
wrong: vocabularies at both sides of each workgroup size and of the largest one it takes,
a last piece of four columns, row counts around a tile of 16 rows, padded and ignored
rows, and logits far apart.  The bound is that of the other bf16 parity tests."""
import numpy as np
import pytest

from tests._parity import TOL, say
from tests.test_gpu_head import _check, _run_head, _synthetic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [4, 36, 512, 516, 1028, 2048, 2052, 4096, 4100, 8196, 12288, 12292, 16388, 24580, 32768, 32772])
@pytest.mark.parametrize("T,B,spread", [(3, 17, 0.0), (2, 1, 80.0), (9, 16, 0.0)])
def test_ce_row(V, T, B, spread):
    say(f"[gpu] ce row V={V} T={T} B={B} spread={spread}")
    lengths = None if B == 1 else np.random.default_rng(V).integers(1, T + 1, size=(B,)).astype(np.int32)
    cfg, wl, y = _synthetic("ce", T, B, 40, V, dtype="bf16", lengths=lengths, seed=V)
    if spread:
        wl.b_fc = (spread * wl.b_fc / np.abs(wl.b_fc).max()).astype(np.float32)
    if B > 1:
        wl.targets[0, 0], wl.targets[0, 1], wl.targets[0, 2] = -1, V, V - 1
    got, ref, _ = _run_head(cfg, wl, y, 0.3, 1)
    _check(got, ref, TOL["bf16"])
