"""Sampling in tiles of every width, operands in place and packed: token counts at the edges of one, two and three tiles, one to
sixteen k-blocks with and without a ragged last one, vocabularies whose last tile is ragged, seeds and temperatures that differ
from case to case.  Draws and scores against the oracle's as in test_gpu_parity.py; test_plan.py checks that each case takes the
tile named here."""
import numpy as np
import pytest

from paper_2602_19362_amd import oapl
from tests.test_gpu_parity import _check_samples, _custom_batch

pytestmark = pytest.mark.gpu

CASES = [   # tokens, hidden size, vocabulary, tile width, operands in place
    (257, 64, 60001, 288, 1), (288, 72, 60001, 288, 1), (289, 128, 60001, 320, 1), (320, 200, 60001, 320, 1),
    (321, 192, 60001, 352, 1), (352, 1024, 60001, 352, 1), (353, 64, 60001, 384, 1), (384, 1024, 60001, 384, 1),
    (513, 136, 30000, 288, 1), (640, 64, 60001, 320, 1), (704, 320, 60001, 352, 1), (1100, 72, 60001, 384, 1),
    (4097, 72, 5003, 384, 0), (4608, 72, 5003, 384, 0), (4097, 72, 300, 256, 0), (8193, 64, 257, 256, 0)]


@pytest.mark.parametrize("T,d,V", [c[:3] for c in CASES])
def test_draws(T, d, V):
    print(T, d, V, flush=True)
    b = _custom_batch("bf16", d=d, V=V, lens=[T], n_groups=1, seed=T + d, beta=1.0)
    temperature, seed = (0.6, 1.0, 1.2)[T % 3], 7 + (T << 33)
    tok, sc, ws = oapl.sample_tokens(b.H, b.W, temperature, seed, want_scores=True)
    assert oapl.read_device_status(ws) == 0
    rows = np.unique(np.concatenate([np.arange(0, T, 5 if T < 1000 else 41), np.arange(T - 34, T)]))    # every lane column
    _check_samples(b.H, b.W, temperature, seed, tok, sc, rows=rows)
