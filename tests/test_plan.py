"""The library's host decisions, host side only: launch grids and plans."""
from tests._plan import ask

INT_MAX = 2 ** 31 - 1


def test_first_launch_indices_fit_32_bits():
    """Sizes up to the documented limit (n_seq * n_groups <= 2^32): the largest thread index and stride of the call's first
    launch fit an int, and few items get a thread (a wavefront) each."""
    sizes = [(4, 1 << 25), (0, INT_MAX), (2, INT_MAX), (1, 1 << 25), (128, 1 << 25), (INT_MAX, 1), (INT_MAX, 2),
             (1 << 16, 1 << 16), (300, 100), (100000, 40), (9000, 1)]
    for (n_seq, n_groups), a in zip(sizes, ask([f"begin {s} {g}" for s, g in sizes])):
        assert a["one"] == 0 or n_seq + n_groups <= 8192
        assert 1 <= a["grid"] * 256 <= INT_MAX, (n_seq, n_groups, a)
        if max(n_seq, 64 * n_groups) <= 1 << 22:
            assert a["grid"] * 256 >= n_seq and a["grid"] * 4 >= n_groups, (n_seq, n_groups, a)
