"""Loss calls whose reference pass comes in parts over the hidden size: parts of unequal length, rows that end inside a k-block,
tokens that end inside a tile, vocabularies of fewer rows than the sample, few rollouts (the call's beginning in the same
launch) and many (in its own).  Tolerances as in test_gpu_parity.py for bf16 inputs; test_plan.py checks the plans."""
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import oracle_full
from tests.test_gpu_parity import _check, _custom_batch, _run

pytestmark = pytest.mark.gpu

CASES = [   # d, V, rollout lengths, what the plan has to say
    (1032, 300, [40, 24], dict(ref_splits=4)),            # 17 k-blocks, the last one of 8 columns
    (1096, 200, [40, 25], dict(ref_splits=2)),            # fewer rows than the sample
    (2048, 257, [65], dict(ref_splits=5)),                # 32 k-blocks: parts of six and seven
    (2104, 1500, [150] * 6 + [101], dict(ref_splits=3)),
    (2048, 9000, [70, 60], dict(ref_splits=8)),
    (1536, 3000, [150] * 20 + [7], dict(ref_splits=5)),
]


@pytest.mark.parametrize("d,V,lens", [c[:3] for c in CASES])
def test_loss(d, V, lens):
    print(d, V, lens, flush=True)
    b = _custom_batch("bf16", d=d, V=V, lens=lens, n_groups=1, seed=d + V, beta=1.0)
    b.H[::3] += 20 * b.W[b.tokens[::3].long()]        # sampled tokens from unlikely to near-certain
    res = _run(b)
    _check(b, res, oracle_full(b), lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3)
    # as many rollouts as do not begin in one launch: the same log-probs, to the bit
    n, dev = 300, b.H.device
    off = torch.clamp(torch.arange(n + 1, device=dev, dtype=torch.int64) * b.T // 64, max=b.T)
    gid = (torch.arange(n, device=dev) % 60).to(torch.int32)
    many = oapl.loss_fwd_bwd(b.H, b.W, b.tokens, b.logq, off, torch.ones(n, device=dev), gid, 60, 1.0)
    assert oapl.read_device_status(many.workspace) == 0 and not oapl.took_two_passes(many.workspace)
    assert torch.equal(res.logprob, many.logprob)
