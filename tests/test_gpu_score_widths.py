"""Scoring in tiles of every width (288 and 352 columns are loads that only half of the wavefronts take part in): token counts at
the edges of one, two and three tiles, with and without ragged k-blocks, and 256 columns with loads that go out early (W of more
than 256 MiB, up to 512 tokens) and spread.  The first two k-blocks are requested in one go and only those behind them between the multiplications, so the
hidden sizes go from one k-block to sixteen.  test_plan.py checks that each case takes the tile named here."""
import numpy as np
import pytest
import torch

from oracle import oapl_oracle as orc
from paper_2602_19362_amd import oapl
from tests._util import f64
from tests.test_gpu_parity import _custom_batch

pytestmark = pytest.mark.gpu

V = 60000
CASES = [(257, 288), (288, 288), (289, 320), (321, 352), (352, 352), (353, 384), (385, 256), (512, 256), (513, 288), (576, 288),
         (650, 352), (704, 352), (864, 288), (1056, 352), (1761, 256), (3201, 256)]     # tokens, tile width
HIDDEN = [64, 72, 192, 200, 256, 320, 328, 1024]     # 1, 2 (ragged), 3, 4 (ragged), 4, 5, 6 (ragged) and 16 k-blocks


EARLY = [(129, 2304), (385, 2296), (512, 2304), (513, 2304)]    # tokens, hidden size; the last is one token too many


@pytest.mark.parametrize("T, d", [(c[0], d) for d in HIDDEN for c in CASES] + EARLY)
def test_scores(T, d):
    print(T, d, flush=True)
    b = _custom_batch("bf16", d=d, V=V, lens=[T], n_groups=1, seed=T + d, beta=1.0)
    lp, lse, ent, ws = oapl.logprob_fwd(b.H, b.W, b.tokens, want_lse=True, want_entropy=True)
    assert oapl.read_device_status(ws) == 0
    plain, _ = oapl.logprob_fwd(b.H, b.W, b.tokens)
    assert torch.equal(lp, plain)
    rows = np.unique(np.concatenate([np.arange(0, T, 7 if T < 1500 else 21), np.arange(T - 40, T)]))     # every lane column, the last tile's edge
    rt = torch.from_numpy(rows).to(b.H.device)
    H, W = f64(b.H[rt]), f64(b.W)
    z = H @ W.T
    ref = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
    assert np.abs(f64(lse[rt]) - ref).max() <= 1e-4      # fp32 sums of exact products over d <= 2304, V = 60000
    assert np.abs(f64(lp[rt]) - (z[np.arange(rows.size), b.tokens[rt].cpu().numpy()] - ref)).max() <= 1e-4
    assert np.abs(f64(ent[rt]) - orc.token_entropy(H, W)).max() <= 2e-3
