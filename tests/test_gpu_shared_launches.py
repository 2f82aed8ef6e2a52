"""Launches that do several steps of a small call: token counts around the 64 of the sweep's first launch and the 4 of the fp32
one, rows of fewer and more 16-byte pieces than the 32 a token's lanes have under way, hidden sizes on both sides of the
line where the steps have launches of their own, vocabularies smaller than the reference sample, an odd number of packed
blocks; both objectives, malformed offsets (the device takes the two-pass schedule) and tokens out of range, which
a later launch than the gather's reports.  Tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import f64, oracle_full
from tests.test_gpu_parity import _check, _custom_batch, _run

pytestmark = pytest.mark.gpu

BF16 = [(8, 64, 40), (248, 65, 255), (256, 127, 256), (264, 129, 257), (320, 200, 700), (1016, 300, 513), (1024, 193, 1500),
        (1032, 193, 1500), (72, 1000, 300)]
F32 = [(1, 1, 3), (33, 5, 65), (64, 63, 1000), (65, 257, 999), (300, 130, 3000)]


@pytest.mark.parametrize("dtype,d,T,V", [("bf16",) + c for c in BF16] + [("f32",) + c for c in F32])
def test_calls(dtype, d, T, V):
    print(dtype, d, T, V, flush=True)
    b = _custom_batch(dtype, d=d, V=V, lens=[T - T // 3, T // 3], n_groups=1, seed=d + T, beta=1.0)
    ref = oracle_full(b)
    tol = dict(lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3) if dtype == "bf16" else \
        dict(lp_tol=1e-5, rel_tol=1e-5, g_rtol=1e-4, g_atol_frac=1e-5)
    res = _run(b)
    _check(b, res, ref, **tol)
    lp_old = (b.logq + 0.01).contiguous()
    g = oapl.grpo_loss_fwd_bwd(b.H, b.W, b.tokens, b.logq, lp_old, b.seq_offsets, b.rewards, b.group_ids, b.n_groups)
    assert oapl.read_device_status(g.workspace) == 0
    assert np.abs(f64(g.logprob) - ref["logprob"]).max() <= tol["lp_tol"]

    # a token out of range: recorded, its log-prob NaN, the others as before
    bad = b.tokens.clone()
    bad[T // 2] = V
    res = oapl.loss_fwd_bwd(b.H, b.W, bad, b.logq, b.seq_offsets, b.rewards, b.group_ids, b.n_groups, b.beta)
    assert oapl.read_device_status(res.workspace) == 9
    lp = f64(res.logprob)
    assert np.isnan(lp[T // 2]) and np.abs(np.delete(lp - ref["logprob"], T // 2)).max(initial=0.0) <= tol["lp_tol"]

    # malformed offsets as well: still the token that is reported, and the loss is NaN
    off = b.seq_offsets.clone()
    off[0] = 1
    res = oapl.loss_fwd_bwd(b.H, b.W, bad, b.logq, off, b.rewards, b.group_ids, b.n_groups, b.beta)
    assert oapl.read_device_status(res.workspace) == 9 and torch.isnan(res.loss).all()
    assert np.isnan(f64(res.logprob)[T // 2])


@pytest.mark.parametrize("T", [384, 700])       # one token tile of the large size; two, and more tiles than compute units
def test_sweeps_on_both_sides_of_early_loads(T):
    b = _custom_batch("bf16", d=512, V=40000, lens=[T - 100, 100], n_groups=1, seed=T, beta=1.0)
    _check(b, _run(b), oracle_full(b), lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3)


# Several panels (384 rows each, two buffers), the call's beginning in one launch.  Whatever closes the sweep, and wherever the bad
# token lies, somebody reports it: an open k_sweep_finish or the fallback.
@pytest.mark.parametrize("objective", ["oapl", "grpo"])
@pytest.mark.parametrize("at", [5, 400, 999])                                   # first, middle and last panel
@pytest.mark.parametrize("closed_by", ["nothing", "rollout", "offsets", "range"])
def test_bad_token_in_several_panels(closed_by, at, objective):
    print(closed_by, at, objective, flush=True)
    d, V, T = 256, 1544, 1000
    b = _custom_batch("bf16", d=d, V=V, lens=[700, 300] if closed_by == "rollout" else [300, 350, 250, 100], n_groups=2, seed=at,
                      beta=1.0)
    if closed_by == "range":       # a row of the first panel whose largest logit is 300 nats above all that the sweep samples
        b.tokens = (b.tokens % 1500).to(torch.int32)
        b.W[1520] = (b.H[10].float() * (300.0 / float((b.H[10].float() ** 2).sum()))).bfloat16()
    ref = oracle_full(b, backward=False)["logprob"]
    bad, off = b.tokens.clone(), b.seq_offsets.clone()
    bad[at] = V
    if closed_by == "offsets":
        off[0] = 1
    args = (b.H, b.W, bad, b.logq)
    rest = (off, b.rewards, b.group_ids, b.n_groups)
    _, rows, buffers = oapl.workspace_bytes_for(T, d, V, b.rewards.shape[0], b.n_groups, oapl.OAPL_BF16, True, 384)
    assert (rows, buffers) == (384, 2)
    if objective == "oapl":
        res = oapl.loss_fwd_bwd(*args, *rest, b.beta, max_panel_rows=384)
    else:
        res = oapl.grpo_loss_fwd_bwd(*args, (b.logq + 0.01).contiguous(), *rest, max_panel_rows=384)
    assert oapl.took_two_passes(res.workspace) == (closed_by != "nothing")
    assert oapl.read_device_status(res.workspace) == 9
    lp = f64(res.logprob)
    assert np.isnan(lp[at]) and np.abs(np.delete(lp - ref, at)).max() <= 2e-2


@pytest.mark.parametrize("d,V", [(8, 300), (128, 300), (136, 700), (512, 1500), (520, 257), (1016, 1500), (1024, 1500)])
def test_sampled_logit_is_the_gathers_to_the_bit(d, V):
    """A sampled token's logit is summed in one order, whichever launch takes it: log-probs do not depend on the number of
    rollouts and prompts (200 x 60 are too many for a beginning in one launch), nor on a bit of it."""
    T = 1000
    few = _custom_batch("bf16", d=d, V=V, lens=[600, 400], n_groups=2, seed=d, beta=1.0)
    few.H[::3] += 20 * few.W[few.tokens[::3].long()]        # sampled tokens from unlikely to near-certain
    n = 200
    off = torch.arange(n + 1, device=few.H.device, dtype=torch.int64) * (T // n)
    gid = (torch.arange(n, device=few.H.device) % 60).to(torch.int32)
    rewards = torch.ones(n, device=few.H.device)
    a = oapl.loss_fwd_bwd(few.H, few.W, few.tokens, few.logq, few.seq_offsets, few.rewards, few.group_ids, 2, 1.0)
    m = oapl.loss_fwd_bwd(few.H, few.W, few.tokens, few.logq, off, rewards, gid, 60, 1.0)
    assert oapl.read_device_status(a.workspace) == oapl.read_device_status(m.workspace) == 0
    assert not oapl.took_two_passes(a.workspace) and not oapl.took_two_passes(m.workspace)
    assert torch.equal(a.logprob, m.logprob)
