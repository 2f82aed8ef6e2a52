"""Batches with more rollouts and prompts than one workgroup looks at in a call's first launch, more rollouts than the
objective takes in one launch and than the workgroup that adds up the loss has threads, and short or empty rollouts; the
sizes just below each line too.  Tolerances as in test_gpu_parity.py."""
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import oracle_full
from tests.test_gpu_parity import _check, _custom_batch, _grpo, _grpo_check, _grpo_inputs, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_seq,n_groups", [(32, 4), (33, 3), (255, 15), (256, 16), (257, 1), (400, 40), (900, 9)])
def test_losses(dtype, n_seq, n_groups):
    print(dtype, n_seq, n_groups, flush=True)
    n_seq = n_seq // n_groups * n_groups
    b = _custom_batch(dtype, d=64, V=300, lens=[i % 4 for i in range(n_seq)], n_groups=n_groups, seed=n_seq, beta=1.0)
    tol = (2e-2, 1e-3, 2e-2, 6e-3) if dtype == "bf16" else (1e-5, 1e-5, 1e-4, 1e-5)
    res = _run(b)
    _check(b, res, oracle_full(b), *tol)
    again = _run(b)
    assert torch.equal(res.loss, again.loss) and torch.equal(res.dW, again.dW)
    # the loss once more, from its parts: NaN-free and fixed whatever the launches
    delta = b.beta * res.seq_logratio.double() - (b.rewards.double() - res.vstar.double()[b.group_ids.long()])
    assert abs((delta ** 2).sum().item() / res.loss.item() - 1) <= 1e-5
    logq, logp_old = _grpo_inputs(b, n_seq)
    res = _grpo(b.H, b.W, b.tokens, logq, logp_old, b.seq_offsets, b.rewards, b.group_ids, n_groups)
    torch.cuda.synchronize()
    _grpo_check(b, logq, logp_old, res, *tol)


def test_more_prompts_than_the_first_launch_has_wavefronts():
    """2^25 prompts for four rollouts, nearly all of them empty: every prompt is visited once (V* is its rollouts' value, or
    NaN), the empty ones make the loss NaN and set the group status, for both objectives."""
    n_groups = 1 << 25
    b = _custom_batch("f32", d=16, V=300, lens=[3, 0, 5, 2], n_groups=1, seed=1, beta=1.0)
    b.group_ids.copy_(torch.tensor([0, n_groups - 1, 12345678, 0], dtype=torch.int32))
    b.rewards.copy_(torch.tensor([1.0, 0.0, 1.0, 1.0]))
    res = oapl.loss_fwd_bwd(b.H, b.W, b.tokens, b.logq, b.seq_offsets, b.rewards, b.group_ids, n_groups, 1.0,
                            backward=False)
    full = torch.nonzero(~torch.isnan(res.vstar)).flatten().cpu()
    assert full.tolist() == [0, 12345678, n_groups - 1]
    assert res.vstar[full.to(b.H.device)].cpu().tolist() == [1.0, 1.0, 0.0]
    assert torch.isnan(res.loss).item() and oapl.read_device_status(res.workspace) == 5
    del res
    logq, logp_old = _grpo_inputs(b, 1)
    res = _grpo(b.H, b.W, b.tokens, logq, logp_old, b.seq_offsets, b.rewards, b.group_ids, n_groups, backward=False)
    assert torch.isnan(res.loss).item() and oapl.read_device_status(res.workspace) == 5
    assert res.advantages.cpu().tolist() == [0.0, 0.0, 0.0, 0.0]
