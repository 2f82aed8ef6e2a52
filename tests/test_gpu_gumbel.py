"""The sampler's Gumbel variates against 64 bits: with one vocabulary entry and zero logits the best score of a row IS the
variate, so 2^20 rows sample the 2^23 words a variate can come from.  Bounds: the error over all words that logf has in the
same formula (9.6e-8 root mean square, 1.88e-6 at most); the hardware's base-2 logarithm must be no worse."""
import numpy as np
import pytest
import torch

from oracle import oapl_oracle as orc
from paper_2602_19362_amd import oapl
from tests._util import f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_variates(dtype):
    T, seed = 1 << 20, 99
    H = torch.zeros(T, 8, dtype=dtype, device="cuda:0")
    tok, score, _ = oapl.sample_tokens(H, H[:1], 1.0, seed, want_scores=True)
    assert not tok.any()
    err = f64(score) - orc.gumbel_noise(np.arange(T), 1, seed)[:, 0]
    print(f"rms {np.sqrt((err ** 2).mean()):.3e} max {abs(err).max():.3e} mean {err.mean():.3e}", flush=True)
    assert np.sqrt((err ** 2).mean()) <= 9.6e-8 and abs(err).max() <= 1.88e-6
