"""fp32 contractions from bf16 parts where a sum has one term, so that nothing hides what a product leaves out."""
import numpy as np
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests._util import f64

pytestmark = pytest.mark.gpu


def _parts(x):
    a = x.bfloat16().float()
    b = (x - a).bfloat16().float()
    return [v.double() for v in (a, b, x - a - b)]


def _mantissas(n):
    """n numbers of [1, 2): those whose later parts are the largest (2^-8 and 2^-17 of the number), and others."""
    x = (1 + torch.arange(1 << 23, dtype=torch.float64) / (1 << 23)).float()
    p = _parts(x)
    worst = ((p[1] * p[2]).abs() / x.double() ** 2).topk(n // 2).indices
    g = torch.Generator().manual_seed(n)
    return torch.cat([x[worst], 1 + torch.rand(n - n // 2, generator=g)])


@pytest.mark.parametrize("T", [3000, 40001])     # 64 x 128 and 128 x 128 tiles
@pytest.mark.parametrize("d", [1, 33])
def test_a_product_goes_into_the_sum_whole(T, d):
    """One vocabulary row: a token's log-sum-exp is its logit.  Rows with one number that is not zero: the logit is one product.
    First products are exact; the others, at most 2^-7 of the whole, are added in seven steps that cut at most a place
    each (7 x 2^-7 of a place of the whole, twice that where the product is just above a power of two), and the sum of both
    is rounded once.  Without x1 y2 and x2 y1 up to 0.97 places."""
    x = _mantissas(T)
    y = x[:1].clone()                            # the largest later parts meet their like
    H = torch.zeros(T, d)
    at = torch.arange(T) % d
    H[torch.arange(T), at] = x
    W = y.expand(1, d).contiguous()
    lse = oapl.logprob_fwd(H.cuda(), W.cuda(), torch.zeros(T, dtype=torch.int32, device="cuda:0"), want_lse=True)[1]
    z = f64(x) * float(y)
    assert (abs(f64(lse) - z) <= (0.5 + 14 / 128 + 0.01) * 2.0 ** (np.floor(np.log2(z)) - 23)).all()
