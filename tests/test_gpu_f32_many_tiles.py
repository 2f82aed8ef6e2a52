"""fp32 calls of more tiles than a launch of 256 threads a workgroup holds in one dimension (2^24)."""
import numpy as np
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import f64
from tests.test_gpu_parity import _check_samples

pytestmark = pytest.mark.gpu


def test_scores_and_samples():
    """T * V / 2^14 > 2^24.  One product a logit; tolerances as in test_gpu_parity.py for fp32 inputs."""
    T, d, V = 1812001, 1, 151936
    g = torch.Generator(device="cuda:0").manual_seed(1)
    H = torch.randn(T, d, generator=g, device="cuda:0")
    W = torch.randn(V, d, generator=g, device="cuda:0")
    tokens = torch.randint(0, V, (T,), generator=g, device="cuda:0").to(torch.int32)
    lp, lse, ws = oapl.logprob_fwd(H, W, tokens, want_lse=True)
    rows = np.unique(np.concatenate([np.arange(0, T, 30011), np.arange(T - 20, T)]))
    at = torch.from_numpy(rows).cuda()
    z = f64(H[at]) @ f64(W).T
    ref = np.log(np.exp(z).sum(1))
    assert abs(f64(lse[at]) - ref).max() <= 1e-5
    assert abs(f64(lp[at]) - (z[np.arange(rows.size), tokens[at].cpu().numpy()] - ref)).max() <= 1e-5
    tok, score, _ = oapl.sample_tokens(H, W, 1.0, 3, want_scores=True, workspace=ws)
    _check_samples(H, W, 1.0, 3, tok, score, rows=rows)
