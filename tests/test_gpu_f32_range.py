"""fp32 contractions over the whole range of fp32: operands whose bf16 parts would be below the least bf16 number, numbers past the
largest, infinities beside the least numbers, and results that the parts' common scale would take out of range.  Tolerances
of the loss as in test_gpu_f32_tiles.py."""
import math

import numpy as np
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import f64, oracle_full
from tests.test_gpu_parity import _check, _custom_batch, _run

pytestmark = pytest.mark.gpu

SHAPES = [   # d, V, rollout lengths, panel cap: 64 x 64 tiles, 128 x 128, 256 x 128, panels that are added to
    (33, 65, [60, 5], 0),
    (67, 994, [150] * 18 + [68], 0),
    (257, 8193, [150] * 6 + [125], 0),
    (21, 700, [70, 60, 0, 62], 64),
]


@pytest.mark.parametrize("to_h,to_w", [(-124, 100), (100, -124), (-120, 120)])
@pytest.mark.parametrize("d,V,lens,cap", SHAPES)
def test_operands_far_from_one(d, V, lens, cap, to_h, to_w):
    """H and W times powers of two: least numbers down to the smallest subnormal, largest past 2^104 (120), where numbers are
    multiplied whole."""
    print(d, V, lens, cap, to_h, to_w, flush=True)
    b = _custom_batch("f32", d=d, V=V, lens=lens, n_groups=1, seed=d + V, beta=1.0)
    b.H *= 2.0 ** to_h
    b.W *= 2.0 ** to_w
    res = _run(b, max_panel_rows=cap or None)
    _check(b, res, oracle_full(b), lp_tol=1e-5, rel_tol=1e-5, g_rtol=1e-4, g_atol_frac=1e-5)
    again = _run(b, max_panel_rows=cap or None)
    assert torch.equal(res.dH, again.dH) and torch.equal(res.dW, again.dW)


def test_gradients_of_improbable_rows():
    """Vocabulary rows of probability 2^-126: their dW as exactly as any.  Logits are 0 and -87 exactly; what is left is the
    rounding of the log-sum-exp (2^-22 of ln 40, as an exponent), of the exponential, of the products and of 64 additions:
    under 1e-5 in all."""
    T, d, V, likely = 64, 8, 64, 40
    b = _custom_batch("f32", d=d, V=V, lens=[T], n_groups=1, seed=3, beta=1.0)
    b.H[:, 0] = 1.0
    b.W.zero_()
    b.W[likely:, 0] = -87.0
    b.tokens %= likely
    ref = oracle_full(b)
    dW = f64(_run(b).dW)[likely:]
    assert 0 < abs(ref["dW"][likely:]).max() < 2.0 ** -110
    assert np.linalg.norm(dW - ref["dW"][likely:]) <= 1e-5 * np.linalg.norm(ref["dW"][likely:])


def test_infinity_times_the_least_numbers():
    """2^-140, which no bf16 number is near, times infinity is infinite, with the product's sign."""
    T, d, V = 70, 8, 130
    g = torch.Generator(device="cuda:0").manual_seed(5)
    H = torch.randn(T, d, generator=g, device="cuda:0")
    W = torch.randn(V, d, generator=g, device="cuda:0")
    W[:, 1] = -2.0 ** -140
    W[7, 1] = 2.0 ** -140
    H[3, 1] = float("inf")
    tok, score, _ = oapl.sample_tokens(H, W, 1.0, 11, want_scores=True)
    assert int(tok[3]) == 7 and float(score[3]) == math.inf
    assert torch.isfinite(score[torch.arange(T, device="cuda:0") != 3]).all()


@pytest.mark.parametrize("T", [70, 40001])      # 64 x 128 and 128 x 128 tiles
def test_results_far_from_one(T):
    """One vocabulary row, so that the log-sum-exp is the logit: one product, rounded once, up to the largest number."""
    h = torch.exp2(torch.linspace(-60.0, 63.9, T, dtype=torch.float64)).float()
    w = torch.tensor([[1.5 * 2.0 ** 63]])
    lse = oapl.logprob_fwd(h[:, None].cuda(), w.cuda(), torch.zeros(T, dtype=torch.int32, device="cuda:0"), want_lse=True)[1]
    z = f64(h) * float(w)
    assert z.max() > 2.0 ** 127 and (abs(f64(lse) - z) <= 0.62 * 2.0 ** (np.floor(np.log2(z)) - 23)).all()
