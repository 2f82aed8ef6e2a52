"""Loss calls small enough for 128 x 128 tiles: tokens, vocabulary and hidden size one short of and past the tile, the
384-row and 256-row blocks it lies in, with large and small tiles mixed between the kernels of one call (k-block counts and
sizes on either side of each rule), under both schedules.  Tolerances as in test_gpu_parity.py."""
import pytest

from tests._util import oracle_full
from tests.test_gpu_parity import _MODE, _check, _custom_batch, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("d,V,T", [(128, 128, 128), (120, 127, 127), (136, 129, 129), (256, 385, 383), (264, 257, 385),
                                   (8, 1544, 513), (392, 770, 640), (1032, 300, 200), (72, 33000, 700), (512, 6000, 64)])
def test_edges(d, V, T, two_pass):
    print(d, V, T, two_pass, flush=True)
    _MODE[0] = "two_pass" if two_pass else "single_sweep"
    try:
        b = _custom_batch("bf16", d=d, V=V, lens=[T // 3, T - T // 3], n_groups=1, seed=d + V + T, beta=1.0)
        _check(b, _run(b), oracle_full(b), lp_tol=2e-2, rel_tol=1e-3, g_rtol=2e-2, g_atol_frac=6e-3)
    finally:
        _MODE[0] = "single_sweep"
