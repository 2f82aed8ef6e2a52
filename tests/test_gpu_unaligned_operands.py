"""bf16 H and W that start at any element of a buffer: same bits as from aligned tensors, through every entry point, where
the kernels read the operands in place and where they are packed, under both schedules."""
import pytest
import torch

from paper_2602_19362_amd import oapl
from tests.test_gpu_parity import _MODE, _custom_batch, _grpo, _grpo_inputs, _run

pytestmark = pytest.mark.gpu


def _at(t, elements):
    """The tensor as a contiguous view `elements` past an aligned address."""
    buf = torch.empty(t.numel() + elements, dtype=t.dtype, device=t.device)
    view = buf[elements:].view_as(t)
    view.copy_(t)
    assert view.is_contiguous() and view.data_ptr() % 16 == 2 * elements % 16
    return view


# in place with small tiles, dH split, one and several panels, the least workspace asked for; packed (ragged rows above 4096 tokens; above 8192)
@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("d,V,lens,cap", [(72, 1003, [40, 20], 0), (264, 1544, [300, 0, 85], 0), (128, 9000, [500, 470], 384),
                                          (128, 9000, [500, 470], 1),
                                          (72, 300, [4000, 100], 0), (64, 300, [8000, 200], 0)])
def test_losses(d, V, lens, cap, two_pass):
    print(d, V, lens, cap, two_pass, flush=True)
    _MODE[0] = "two_pass" if two_pass else "single_sweep"
    try:
        b = _custom_batch("bf16", d=d, V=V, lens=lens, n_groups=1, seed=d + V, beta=1.0)
        logq, logp_old = _grpo_inputs(b, d)
        H, W = b.H, b.W
        results = []
        for h, w in ((0, 0), (1, 0), (0, 4), (7, 3)):
            b.H, b.W = (_at(H, h) if h else H), (_at(W, w) if w else W)
            r = _run(b, max_panel_rows=cap or None)
            assert oapl.read_device_status(r.workspace) == 0
            g = _grpo(b.H, b.W, b.tokens, logq, logp_old, b.seq_offsets, b.rewards, b.group_ids, 1)
            results.append(r[:6] + g[:5])
        assert torch.isfinite(results[0][5]).all()
        for other in results[1:]:
            assert all(torch.equal(x, y) for x, y in zip(results[0], other))
    finally:
        _MODE[0] = "single_sweep"


@pytest.mark.parametrize("T,d,V", [(1, 8, 300), (64, 128, 700), (129, 72, 1544), (400, 64, 60000), (4097, 72, 300)])
def test_scores_samples_and_the_call_without_workspace(T, d, V):
    print(T, d, V, flush=True)
    b = _custom_batch("bf16", d=d, V=V, lens=[T], n_groups=1, seed=T + d, beta=1.0)

    def calls(H, W):
        out = oapl.logprob_fwd(H, W, b.tokens, want_lse=True, want_entropy=True)[:-1]
        out += oapl.sample_tokens(H, W, 0.8, 11, want_scores=True)[:-1]
        if T * V < 1 << 20:
            new = lambda *s: torch.empty(*s, device=H.device)
            outs = (new(1), new(T), new(1), new(1), torch.empty_like(b.H), new(V, d))
            oapl.loss_fwd_bwd_noalloc(H, W, b.tokens, b.logq, b.seq_offsets, b.rewards, b.group_ids, 1, 1.0, *outs)
            out += outs
        torch.cuda.synchronize()
        return out

    want = calls(b.H, b.W)
    assert torch.isfinite(want[0]).all()
    for h, w in ((1, 5), (2, 0), (0, 1)):
        assert all(torch.equal(x, y) for x, y in zip(want, calls(_at(b.H, h) if h else b.H, _at(b.W, w) if w else b.W)))
