"""Loss calls whose sweep, recompute and dH take tiles of 256 to 352 columns: tokens at the edges of one, two and three tiles
(those of 288 and 352 end in the middle of the 64-token blocks that dW walks), ragged vocabulary and hidden size, both
schedules.  Tolerances as in test_gpu_parity.py; test_plan.py checks that each case takes the width named here."""
import pytest
import torch

from tests._util import oracle_full
from tests.test_gpu_parity import _MODE, _check, _custom_batch, _run

pytestmark = pytest.mark.gpu

D, V = 1000, 50003
CASES = [(257, 320), (320, 320), (385, 256), (512, 256), (513, 288), (576, 288), (577, 320), (640, 320), (641, 352), (704, 352),
         (777, 288), (961, 352)]      # tokens, tile width


@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("T", [c[0] for c in CASES])
def test_widths(T, two_pass):
    print(T, two_pass, flush=True)
    _MODE[0] = "two_pass" if two_pass else "single_sweep"
    try:
        b = _custom_batch("bf16", d=D, V=V, lens=[T // 3, T - T // 3], n_groups=1, seed=T, beta=1.0)
        res = _run(b)
        _check(b, res, oracle_full(b), lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3)
        again = _run(b)
        assert torch.equal(res.dH, again.dH) and torch.equal(res.dW, again.dW)
    finally:
        _MODE[0] = "single_sweep"
