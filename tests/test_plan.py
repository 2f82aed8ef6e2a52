"""The library's host decisions, host side only: launch grids and plans."""
import pytest

from paper_2602_19362_amd import oapl
from tests import (test_gpu_dh_splits, test_gpu_f32_parts, test_gpu_f32_tiles, test_gpu_loss_widths, test_gpu_ref_splits,
                   test_gpu_row_walks, test_gpu_sample_widths, test_gpu_score_widths, test_gpu_small_tiles)
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


def test_few_workgroups_hand_the_loss_over():
    """A hand-over costs a fence and a counter per rollout (2048 rollouts: 134 us against 13 in two launches)."""
    sizes = [0, 1, 8, 32, 33, 64, 2048]
    for n, a in zip(sizes, ask([f"objective {n}" for n in sizes])):
        assert a["grid"] == max(n, 1) and a["hand_over"] <= 32


def test_operands_that_are_not_aligned_have_room_for_an_aligned_copy():
    """The kernels that read bf16 W and H in place want them 16-byte aligned: a call whose operands are not copies them
    first, within the workspace the library asks for; one whose operands are needs no such space."""
    for T, d, V in [(1, 8, 8), (64, 4096, 151936), (777, 2048, 3000), (8192, 64, 1000), (4000, 72, 5003), (0, 64, 100)]:
        for bwd in (0, 1):
            nbytes = oapl.workspace_bytes(T, d, V, 1, 1, oapl.OAPL_BF16, bool(bwd))
            plans = ask([f"plan {T} {d} {V} 1 {bwd} 0 {u} -1" for u in range(4)])
            assert [(p["rc"], p["rows"], p["copies"], p["have"]) for p in plans] == [(0, 1, u, nbytes) for u in range(4)]
            assert nbytes >= plans[0]["total"] + 2 * V * d + 2 * T * d
    # packed operands are copies already, and fp32 takes any address
    for q in ("plan 8193 64 1000 1 1 0 3 -1", "plan 4097 72 1000 1 1 0 3 -1", "plan 300 72 1000 0 1 0 0 -1"):
        assert ask([q])[0]["copies"] == 0


def test_small_panels_leave_the_scoring_pass_its_workgroups():
    """The two-pass schedule's scoring pass covers the whole batch whatever the panels: a cap on the panel does not cut its
    vocabulary splits (its partial sums have the panel buffers for their space)."""
    for T, d, V, cap in [(16411, 4096, 151936, 6144), (16411, 4096, 151936, 384), (30011, 5120, 151936, 6144),
                         (3000, 4096, 151936, 384), (3000, 1024, 32000, 768), (1000, 72, 9001, 1), (140897, 4096, 151936, 768)]:
        full, capped = ask([f"plan {T} {d} {V} 1 1 {c} 0 -1" for c in (0, cap)])
        assert capped["rc"] == 0 and capped["panel"] < full["panel"] and capped["have"] < full["have"]
        assert (capped["fwd_tile"], capped["fwd_splits"]) == (full["fwd_tile"], full["fwd_splits"])


def test_a_few_missing_bytes_cost_a_few_splits():
    """Scoring and sampling of few tokens, where a workgroup is a split, on less than the workspace asked for."""
    for T, d, V in [(64, 4096, 151936), (1, 8, 60000), (120, 2048, 151936)]:
        full = ask([f"plan {T} {d} {V} 1 0 0 0 -1"])[0]
        splits = max(full["fwd_splits"], full["smp_splits"])
        for part in (0.99, 0.75, 0.5, 0.1):
            have = int(full["total"] - (1 - part) * splits * T * 12)
            p = ask([f"plan {T} {d} {V} 1 0 0 0 {have}"])[0]
            assert p["rc"] == 0 and p["total"] <= have
            assert min(p["fwd_splits"], p["smp_splits"]) >= part * splits - 512 / T - 2, (T, part, full, p)


@pytest.mark.parametrize("dtype,cases", [
    (oapl.OAPL_BF16, [(sum(lens), d, V, cap, want) for d, V, lens, cap, want in test_gpu_dh_splits.CASES]),
    (oapl.OAPL_BF16, [(T, d, V, 0, want) for d, V, T, want in test_gpu_small_tiles.CASES]),
    (oapl.OAPL_F32, [(sum(lens), d, V, cap, want) for d, V, lens, cap, want in test_gpu_f32_tiles.CASES]),
    (oapl.OAPL_F32, [(sum(lens), d, V, cap, want) for d, V, lens, cap, want in test_gpu_f32_parts.CASES]),
    (oapl.OAPL_BF16, [(sum(lens), d, V, 0, want) for d, V, lens, want in test_gpu_ref_splits.CASES])],
    ids=["dh_splits", "small_tiles", "f32_tiles", "f32_parts", "ref_splits"])
def test_gpu_cases_have_the_plans_they_name(dtype, cases):
    """A change of the time models must not empty the GPU tests of the kernels they are there for."""
    plans = ask([f"plan {T} {d} {V} {dtype} 1 {cap} 0 -1" for T, d, V, cap, _ in cases])
    for (T, d, V, cap, want), plan in zip(cases, plans):
        assert plan["rc"] == 0 and {k: plan[k] for k in want} == want, (T, d, V, cap, plan)


def test_loss_tiles_are_as_wide_as_the_tokens_need():
    """The widths that the GPU test of the loss tiles names; small sweeps, packed operands and capped panels keep 384."""
    d, V = test_gpu_loss_widths.D, test_gpu_loss_widths.V
    plans = ask([f"plan {T} {d} {V} 1 1 0 0 -1" for T, _ in test_gpu_loss_widths.CASES])
    assert [p["width"] for p in plans] == [w for _, w in test_gpu_loss_widths.CASES]
    for q in ("plan 100 4096 151936 1 1 0 0 -1", "plan 8193 4096 151936 1 1 0 0 -1", "plan 777 1000 50003 1 1 384 0 -1",
              "plan 0 1000 50003 1 1 0 0 -1"):
        assert ask([q])[0]["width"] == 384, q


@pytest.mark.parametrize("T,d,V,width", [
    (3678, 1624, 12314, 384), (2849, 1160, 86626, 384), (2116, 936, 28945, 384),      # 1 .. 4 % by the model
    (3230, 680, 21976, 384), (917, 816, 21429, 320), (393, 584, 26488, 256),          # dH in small tiles
    (3989, 2688, 2364, 256), (3495, 2288, 138621, 320), (5081, 3712, 25440, 352)])
def test_loss_tiles_are_narrower_only_where_that_is_sure_to_pay(T, d, V, width):
    assert ask([f"plan {T} {d} {V} 1 1 0 0 -1"])[0]["width"] == width


def test_scoring_tiles_are_as_wide_as_the_tokens_need():
    """The widths that the GPU test of the scoring tiles names."""
    width = {2: 256, 3: 320, 4: 384, 5: 288, 6: 352}       # FwdTile
    for d in test_gpu_score_widths.HIDDEN:
        plans = ask([f"plan {T} {d} {test_gpu_score_widths.V} 1 0 0 0 -1" for T, _ in test_gpu_score_widths.CASES])
        assert [width[p["fwd_tile"]] for p in plans] == [w for _, w in test_gpu_score_widths.CASES]


def test_loads_go_out_early_where_w_comes_from_memory():
    """256-wide tiles of up to 512 tokens, over a W that is larger than the memory-side cache."""
    def early(T, d, V):
        return ask([f"plan {T} {d} {V} 1 0 0 0 -1"])[0]["fwd_early"]
    cases = test_gpu_score_widths
    assert [early(T, d, cases.V) for T, d in cases.EARLY] == [1, 1, 1, 0]
    assert not any(early(T, d, cases.V) for T, _ in cases.CASES for d in cases.HIDDEN)
    # calls on small heads: 8 .. 9 % slower with early loads
    assert [early(T, d, V) for T, d, V in [(192, 2048, 5500), (507, 1024, 351), (410, 2048, 2100), (200, 4096, 32000)]] == [0] * 4
    assert early(200, 4096, 32769) == early(200, 2048, 151936) == 1



@pytest.mark.parametrize("d, V", [(64, 300), (64, 3951), (256, 1544), (256, 15000), (512, 3884), (1024, 2162), (1024, 8192)])
def test_a_shared_launch_spreads_dw_over_the_dies(d, V):
    """Each of dW's tiles once, no XCD with more than its eighth of them."""
    a = ask([f"shared_dw {d} {V}"])[0]
    assert a["once"] == a["tiles"] and a["most"] == (a["tiles"] + 7) // 8


@pytest.mark.parametrize("T, d, V, split", [
    (1, 8, 1, False), (64, 64, 192, False), (1000, 256, 1280, False), (1000, 256, 1344, True),
    (3000, 256, 1544, False), (2000, 512, 2000, False), (8000, 256, 9088, False), (8000, 256, 9152, True), (8000, 256, 15000, True)])
def test_dh_is_split_where_its_walk_outlasts_dws(T, d, V, split):
    """In the launch that both share, on both sides of the line."""
    p = ask([f"plan {T} {d} {V} 1 1 0 0 -1"])[0]
    assert p["rc"] == 0 and p["dh_small"] and p["small_dw"] and (p["dh_splits"] > 1) == split


@pytest.mark.parametrize("rows", [128, 256, 320])
@pytest.mark.parametrize("V", [1, 16, 127, 300, 5003, 32000, 60000, 151936, 2 ** 21])
def test_balanced_walks_cover_the_vocabulary(V, rows):
    """Every row once, in as few tiles as its workgroup needs, and no workgroup with over 32 rows more than another."""
    for per_cu in (1, 2, 3):
        n = min(per_cu * 256, (V + rows - 1) // rows)
        a = ask([f"walks {V} {n} {rows}"])[0]
        assert a["wrong"] == 0 and a["end"] == V and a["most"] - a["least"] <= 32


def test_few_tokens_have_the_walks_they_need():
    """What the GPU test of the walks names, scoring and sampling alike."""
    for d, V, tokens, walks in test_gpu_row_walks.CASES:
        for T, want in zip(tokens, walks, strict=True):
            p = ask([f"plan {T} {d} {V} 1 0 0 0 -1"])[0]
            for even, tall in ((p["even"], p["tall"]), (p["smp_even"], p["smp_tall"])):
                assert "o" * p["once"] + "e" * even + "t" * tall == want, (T, d, V, p)


@pytest.mark.parametrize("T,d,V,even", [
    (64, 1000, 104857, 0), (48, 1800, 101000, 0), (64, 1000, 121217, 1), (64, 1000, 121216, 0), (64, 1000, 130944, 1),
    (17, 1000, 130945, 0), (1, 1000, 151936, 0), (16, 1000, 101632, 0), (1, 1000, 101633, 1), (16, 1000, 140672, 1),
    (16, 1000, 140673, 0), (16, 480, 104857, 0), (16, 480, 104858, 1), (16, 320, 122000, 1), (17, 1000, 104858, 0),
    (128, 1000, 127926, 1), (65, 1000, 127927, 0), (128, 1000, 138412, 0), (128, 1000, 138413, 1), (128, 1024, 131073, 1),
    (200, 760, 84900, 0), (200, 776, 108100, 0), (200, 776, 108101, 1), (200, 1152, 113777, 0), (200, 1152, 113778, 1),
    (256, 128, 114688, 0), (256, 128, 114689, 1), (256, 512, 65000, 1)])
def test_walks_are_even_where_that_is_faster(T, d, V, even):
    """On both sides of each line: 3.1, 3.7, 4 and 4.3 whole tiles per CU, W of 96, 160, 244, 250 and 264 MiB, rows of whole
    lines and others, 448 rows per CU."""
    p = ask([f"plan {T} {d} {V} 1 0 0 0 -1"])[0]
    assert (p["even"], p["smp_even"], p["once"]) == (even, even, 0), p


@pytest.mark.parametrize("T,d,V,even", [
    (128, 384, 65536, 1), (128, 384, 65537, 0), (65, 64, 98304, 0), (128, 64, 98305, 1), (128, 392, 83200, 1)])
def test_draws_on_small_hidden_sizes_take_whole_tiles(T, d, V, even):
    """Two to three tiles per CU, up to d = 384; scoring does not."""
    p = ask([f"plan {T} {d} {V} 1 0 0 0 -1"])[0]
    assert (p["even"], p["smp_even"], p["once"]) == (1, even, 0), p


def test_sampling_tiles_are_as_wide_as_the_tokens_need():
    """The widths that the GPU test of the sampling tiles names."""
    width = {2: 256, 3: 320, 4: 384, 5: 288, 6: 352}       # FwdTile
    cases = test_gpu_sample_widths
    for T, d, V, w, rows in cases.CASES:
        p = ask([f"plan {T} {d} {V} 1 0 0 0 -1"])[0]
        assert (width[p["smp_tile"]], p["rows"]) == (w, rows), (T, d, V, p)


@pytest.mark.parametrize("tiles", [1, 8, 9, 1187, 2 ** 22, 2 ** 22 + 1, 2 ** 24 + 1187, 2 ** 30])
def test_fp32_launches_hold_every_tile(tiles):
    """Up to the tiles of the most tokens and the largest vocabulary: fewer threads than 2^32 in a dimension, a multiple of eight
    workgroups in a row (XCDs take turns), and no more idle ones than a row of them."""
    a = ask([f"f32grid {tiles}"])[0]
    assert a["tiles"] >= tiles and a["most"] < 2 ** 32 and a["rest"] == 0
    assert a["tiles"] - tiles < (8 if tiles <= 2 ** 22 else 2 ** 22)


@pytest.mark.parametrize("T,V,rollouts,together", [
    (5000, 64, 1, 0), (2048, 64, 1, 0), (513, 64, 1, 0), (512, 64, 1, 1), (32, 8192, 4, 0), (16, 8192, 1, 1),
    (256, 1024, 8, 1), (257, 1024, 64, 0), (256, 1024, 7, 0), (256, 1024, 1, 0), (128, 1024, 1, 1), (100, 64, 0, 1)])
def test_log_probs_are_finished_with_the_objective_where_that_is_short(T, V, rollouts, together):
    """Rounds of 256 tokens at V = 64, 64 at 1024 and 8 at 8192, one after the other if one rollout has them."""
    a = ask([f"finish {T} {V} {rollouts}"])[0]
    assert a == dict(ok=1, together=together)
