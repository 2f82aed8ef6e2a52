"""The dH contraction with several workgroups per tile: token counts around the 64-token k-blocks of dW and the token
tile, ragged hidden sizes and vocabularies, from too few k-blocks to split up to tens of splits, operands in place and
packed, one panel and a ragged last panel.  Tolerances as in test_gpu_parity.py; test_plan.py checks that the plan of each
case is the one named here."""
import pytest
import torch

from tests._util import oracle_full
from tests.test_gpu_parity import _MODE, _check, _custom_batch, _run

pytestmark = pytest.mark.gpu


CASES = [   # d, V, rollout lengths, panel cap, what the plan has to say
    (8, 200, [40, 25], 0, dict(rows=1, dh_splits=1)),                   # 4 k-blocks: one split
    (264, 1001, [64, 0, 1, 62], 0, dict(rows=1, dh_splits=4)),          # a ragged second m-tile, two k-blocks of tokens with a ragged tail
    (72, 9000, [383, 1], 0, dict(rows=1, dh_splits=29)),                # 141 k-blocks for one tile: many splits, exactly one token tile
    (520, 20011, [300, 85], 0, dict(rows=1, dh_splits=12)),             # one token past the tile
    (5584, 6801, [100, 45], 0, dict(rows=1, dh_small=1, dh_splits=5, dh_groups=440)),   # small tiles, two workgroups per CU
    (136, 5003, [500, 470], 384, dict(rows=1, panel=384, dh_splits=1)),   # small panels: no room for partial sums
    (72, 1001, [4000, 100], 0, dict(rows=0, dh_splits=1)),              # packed operands, a W too small to lie partial sums in
    (72, 20011, [4000, 100], 0, dict(rows=0, panel=4224, dh_splits=4)),   # the partial sums lie in the packed copy of W
    (72, 5000, [12000, 300, 0, 500], 0, dict(rows=0, panel=12288, dh_splits=8)),   # ... those of a ragged second panel
    (72, 5000, [12500, 300], 0, dict(rows=0, panel=12288, dh_splits=8)),   # ... where the device chooses the two-pass schedule
]


@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("d,V,lens,cap", [c[:4] for c in CASES])
def test_split_tiles(d, V, lens, cap, two_pass):
    print(d, V, lens, cap, two_pass, flush=True)
    _MODE[0] = "two_pass" if two_pass else "single_sweep"
    try:
        b = _custom_batch("bf16", d=d, V=V, lens=lens, n_groups=2 if len(lens) % 2 == 0 else 1, seed=d + V, beta=1.0)
        res = _run(b, max_panel_rows=cap or None)
        _check(b, res, oracle_full(b), lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3,
               fallback=max(lens) > (cap or 12288))
        again = _run(b, max_panel_rows=cap or None)
        assert torch.equal(res.dH, again.dH) and torch.equal(res.dW, again.dW)
    finally:
        _MODE[0] = "single_sweep"
