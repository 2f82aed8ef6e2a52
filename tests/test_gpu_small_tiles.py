"""Loss calls small enough for 128 x 128 tiles: tokens, vocabulary and hidden size one short of and past the tile, the
384-row and 256-row blocks it lies in, with large and small tiles mixed between the kernels of one call (k-block counts and
sizes on either side of each rule; rings of four LDS stages and, where there are more tiles than compute units, of two),
under both schedules.  Tolerances as in test_gpu_parity.py; test_plan.py checks what is said about the plans."""
import pytest

from tests._util import oracle_full
from tests.test_gpu_parity import _MODE, _check, _custom_batch, _run

pytestmark = pytest.mark.gpu


ALL = dict(small_sweep=1, small_dw=1, dh_small=1)
CASES = [(128, 128, 128, ALL), (120, 127, 127, ALL), (136, 129, 129, ALL), (256, 385, 383, ALL), (264, 257, 385, ALL),
         (8, 1544, 513, ALL), (392, 770, 640, ALL), (1032, 300, 200, ALL), (512, 6000, 64, ALL),
         (72, 33000, 700, dict(ALL, sweep_groups=1548, dw_groups=258)),
         (1696, 102, 2549, dict(ALL, dh_splits=1, dh_groups=280)), (2056, 130, 2101, dict(ALL, dh_splits=1, dh_groups=289))]


@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("d,V,T", [c[:3] for c in CASES])
def test_edges(d, V, T, two_pass):
    print(d, V, T, two_pass, flush=True)
    _MODE[0] = "two_pass" if two_pass else "single_sweep"
    try:
        b = _custom_batch("bf16", d=d, V=V, lens=[T // 3, T - T // 3], n_groups=1, seed=d + V + T, beta=1.0)
        _check(b, _run(b), oracle_full(b), lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3)
    finally:
        _MODE[0] = "single_sweep"
