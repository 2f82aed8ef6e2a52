"""Scoring and sampling at the edges of every tile the dispatch can choose: one token up to just past each tile's
width, vocabularies a row short of and past a tile, hidden sizes whose last k-block is ragged, both operand layouts
(in place and packed).  Tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import oapl_oracle as orc
from paper_2602_19362_amd import oapl
from tests._util import f64
from tests.test_gpu_parity import _check_samples, _custom_batch

pytestmark = pytest.mark.gpu


def _check(T, d, V, rows):
    print(f"T={T} d={d} V={V}", flush=True)
    b = _custom_batch("bf16", d=d, V=V, lens=[T], n_groups=1, seed=T + d + V, beta=1.0)
    lp, lse, ent, ws = oapl.logprob_fwd(b.H, b.W, b.tokens, want_lse=True, want_entropy=True)
    tok, sc, ws2 = oapl.sample_tokens(b.H, b.W, 0.9, 77, want_scores=True)
    torch.cuda.synchronize()
    assert oapl.read_device_status(ws) == 0 and oapl.read_device_status(ws2) == 0
    lp2, _ = oapl.logprob_fwd(b.H, b.W, b.tokens)
    assert torch.equal(lp, lp2)
    r = np.arange(T) if T <= rows else np.unique(np.concatenate(
        [np.arange(8), np.arange(T - 8, T), np.linspace(0, T - 1, rows).astype(np.int64)]))
    rt = torch.from_numpy(r).to(b.H.device)
    H, W = f64(b.H[rt]), f64(b.W)
    z = H @ W.T
    ref_lse = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
    ref_lp = z[np.arange(r.size), b.tokens[rt].cpu().numpy()] - ref_lse
    assert np.abs(f64(lse[rt]) - ref_lse).max() <= 1e-4      # fp32 sums of exact products over d <= 1024, V <= 60000
    assert np.abs(f64(lp[rt]) - ref_lp).max() <= 1e-4
    assert np.abs(f64(ent[rt]) - orc.token_entropy(H, W)).max() <= 2e-3
    _check_samples(b.H, b.W, 0.9, 77, tok, sc, rows=r)


@pytest.mark.parametrize("V", [127, 129, 700])
def test_small_token_counts(V):
    for T, d in ((1, 8), (2, 72), (63, 128), (64, 200), (65, 64), (127, 72), (128, 64), (129, 136), (256, 64), (257, 72)):
        _check(T, d, V, 300)


# the 64- and 128-token tiles, which hold a whole block's fragments, over three and more k-blocks, a ragged last one among them
@pytest.mark.parametrize("T,d", [(1, 192), (33, 200), (64, 320), (65, 192), (100, 328), (128, 200), (128, 1024)])
def test_small_tiles_over_many_blocks(T, d):
    _check(T, d, 700, 300)


# 256-, 320- and 384-wide tiles: which one is taken depends on how the tiles divide over 256 compute units
@pytest.mark.parametrize("T,d,V", [(300, 64, 60000), (640, 72, 60000), (641, 64, 60000), (1100, 72, 60000)])
def test_wide_tiles(T, d, V):
    _check(T, d, V, 96)


# packed operands: ragged rows above 4096 tokens, whole lines above 8192
@pytest.mark.parametrize("T,d,V", [(4096, 72, 300), (4097, 72, 300), (8192, 64, 300), (8193, 64, 300)])
def test_packed_operands(T, d, V):
    _check(T, d, V, 400)
