"""Scoring and sampling of up to 256 tokens.  Over a W that is read past the caches (more than 288 MiB, whole 128-byte lines): token
counts at the edges of the three widths, walks of one to three tiles of unequal heights, tiles of 256 and of 320 rows, hidden
sizes whose rows are a multiple of 4 KiB apart (walks over k that start at any block) and others, and one just under the line.  Over
others: tiles of 320 rows, with and without a ragged last k-block, and whole tiles beside even shares.  Tolerances as in
test_gpu_forward_tiles.py; test_plan.py checks that each case has the walks named here."""
import numpy as np
import pytest
import torch

from oracle import oapl_oracle as orc
from paper_2602_19362_amd import oapl
from tests._util import f64
from tests.test_gpu_parity import _check_samples, _custom_batch

pytestmark = pytest.mark.gpu


CASES = [   # hidden size, vocabulary, tokens, what the plan of each has to say: W read once, even shares, 320 rows
    (2048, 73733, [1, 64, 65, 128, 129, 256], ["oe", "oe", "oe", "oe", "oet", "oet"]),       # 289 rows per CU: one tile of 320
    (2048, 120001, [17, 100, 200], ["oe", "oe", "oe"]),       # 469: two of 256
    (1088, 151936, [64, 128, 192], ["oe", "oe", "oet"]),      # 17 k-blocks, two of 320
    (4096, 36865, [1, 128, 256], ["oe", "oe", "oe"]),         # 145 rows per CU
    (4096, 36863, [63, 255], ["", "e"]),                      # 288 MiB less two rows
    (1000, 73733, [129, 200, 256], ["et", "et", "et"]),       # 16 k-blocks, the last one ragged: one tile of 320
    (1000, 151936, [64, 256], ["", "et"]),                    # two of 320 over a W that no cache holds
    (512, 72000, [200], ["et"]),
    (72, 151936, [16, 250], ["", "et"]),                      # two k-blocks
    (1000, 125000, [64], ["e"]),
    (1000, 133169, [128], [""]),
    (512, 91001, [130, 200], ["", ""]),
    (512, 120001, [200], ["e"]),
]


@pytest.mark.parametrize("d, V, tokens", [c[:3] for c in CASES])
def test_calls(d, V, tokens):
    for T in tokens:
        print(T, d, V, flush=True)
        b = _custom_batch("bf16", d=d, V=V, lens=[T], n_groups=1, seed=T + d, beta=1.0)
        lp, lse, ent, ws = oapl.logprob_fwd(b.H, b.W, b.tokens, want_lse=True, want_entropy=True)
        tok, sc, ws2 = oapl.sample_tokens(b.H, b.W, 0.9, 77, want_scores=True)
        assert oapl.read_device_status(ws) == 0 and oapl.read_device_status(ws2) == 0
        assert torch.equal(lp, oapl.logprob_fwd(b.H, b.W, b.tokens)[0])
        r = np.unique(np.concatenate([np.arange(min(T, 4)), np.linspace(0, T - 1, 20).astype(np.int64)]))
        rt = torch.from_numpy(r).to(b.H.device)
        H, W = f64(b.H[rt]), f64(b.W)
        z = H @ W.T
        ref = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
        assert np.abs(f64(lse[rt]) - ref).max() <= 1e-4      # fp32 sums of exact products over d <= 4096
        assert np.abs(f64(lp[rt]) - (z[np.arange(r.size), b.tokens[rt].cpu().numpy()] - ref)).max() <= 1e-4
        assert np.abs(f64(ent[rt]) - orc.token_entropy(H, W)).max() <= 2e-3
        _check_samples(b.H, b.W, 0.9, 77, tok, sc, rows=r)
