"""fp32 contractions from bf16 parts: the 256 x 128 gradient tiles at their edges (one row, one column past a tile, k that ends
inside a stage, splits, panels that are added to), and numbers whose parts are not those of an ordinary one.  Tolerances of the
loss as in test_gpu_f32_tiles.py; test_plan.py checks that the plan of each case is the one named here."""
import numpy as np
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import f64, oracle_full
from tests.test_gpu_parity import _check, _custom_batch, _run

pytestmark = pytest.mark.gpu

CASES = [   # d, V, rollout lengths, panel cap, what the plan has to say
    (257, 8193, [150] * 6 + [125], 0, dict(wide_dh=17, wide_dw=2)),
    (641, 8321, [150] * 8 + [100], 0, dict(wide_dh=7, wide_dw=1)),
    (513, 8193, [150] * 33 + [50], 0, dict(panel=4096, wide_dw=1)),
]


@pytest.mark.parametrize("d,V,lens,cap", [c[:4] for c in CASES])
def test_wide_gradient_tiles(d, V, lens, cap):
    print(d, V, lens, cap, flush=True)
    b = _custom_batch("f32", d=d, V=V, lens=lens, n_groups=1, seed=d + V, beta=1.0)
    res = _run(b, max_panel_rows=cap or None)
    _check(b, res, oracle_full(b), lp_tol=1e-5, rel_tol=1e-5, g_rtol=1e-4, g_atol_frac=1e-5)
    again = _run(b, max_panel_rows=cap or None)
    assert torch.equal(res.dH, again.dH) and torch.equal(res.dW, again.dW)


@pytest.mark.parametrize("d", [5, 40])
def test_numbers_at_the_ends_of_the_range(d):
    """Numbers past the largest bf16 (their first part is infinite), infinite ones and NaN: logits as fp32 products give
    them.  Infinity times a number is infinite with the product's sign whatever the number's later parts are, times zero NaN."""
    T, V = 70, 130
    g = torch.Generator(device="cuda:0").manual_seed(d)
    H = torch.randn(T, d, generator=g, device="cuda:0").abs() + 0.01
    W = torch.randn(V, d, generator=g, device="cuda:0")
    tokens = torch.arange(T, device="cuda:0").to(torch.int32)
    big = torch.finfo(torch.float32).max
    H[:, 1] = 2.0 ** -126             # (numbers with all their bits: test_gpu_f32_range.py)
    W[:, 1] = big * (1 - 2.0 ** -9 * torch.rand(V, generator=g, device="cuda:0"))
    assert (W[:, 1].to(torch.bfloat16).isinf()).any() and W[:, 1].isfinite().all()
    W[100, 2] = -float("inf")         # a logit of -inf for every token: never drawn, no part of any sum
    H[3, 0] = float("inf")            # logits of +inf and -inf
    H[4, 3] = float("nan")
    H[5, 2] = 0.0                     # 0 * -inf
    lp, lse, ent, _ = oapl.logprob_fwd(H, W, tokens, want_lse=True, want_entropy=True)
    torch.cuda.synchronize()
    z = f64(H) @ f64(W).T
    ok = np.array([t not in (3, 4, 5) for t in range(T)])
    assert np.isneginf(z[ok][:, 100]).all() and np.isfinite(np.delete(z[ok], 100, axis=1)).all()
    ref = np.log(np.exp(z[ok]).sum(1))
    assert abs(f64(lse)[ok] - ref).max() <= 1e-5
    assert abs(f64(lp)[ok] - (z[ok][np.arange(T)[ok] >= 0, np.arange(T)[ok]] - ref)).max() <= 1e-5
    assert np.isfinite(f64(ent)[ok]).all()
    assert not np.isfinite(f64(lse)[~ok]).any()


@pytest.mark.parametrize("off", [[0, 40, 70], [5, 40, 70], [0, 60, 30], [50, 10, 20], [0, 200, 70], [-3, 10, 66], [0, 0, 0]])
@pytest.mark.parametrize("d,V", [(40, 130), (40, 6000)])      # finished in the objective's launch and in one of its own
def test_every_token_has_its_log_prob_whatever_the_offsets(d, V, off):
    T = 70
    b = _custom_batch("f32", d=d, V=V, lens=[40, 30], n_groups=1, seed=V, beta=1.0)
    off = torch.tensor(off, dtype=torch.int64, device=b.H.device)
    res = oapl.loss_fwd_bwd(b.H, b.W, b.tokens, b.logq, off, b.rewards, b.group_ids, 1, 1.0)
    assert (oapl.read_device_status(res.workspace) != 0) == (off.tolist() != [0, 40, 70])
    z = f64(b.H) @ f64(b.W).T
    ref = z[np.arange(T), b.tokens.cpu().numpy()] - np.log(np.exp(z).sum(1))
    assert abs(f64(res.logprob) - ref).max() <= 1e-5
