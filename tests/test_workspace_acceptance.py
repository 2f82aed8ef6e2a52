"""Workspace sizes that have always been enough stay enough: byte counts written out here, from plans with fewer partial
sums per token than today's.  Host side only: without a GPU an accepted call ends in the HIP error of its first launch,
a refused one in the workspace error, so on a machine with a GPU (where the pointers would be used) this is skipped."""
import pytest
import torch

from paper_2602_19362_amd import oapl

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="the pointers are stand-ins")
X = 0x10000
ERR_WORKSPACE, ERR_HIP, ERR_SCRATCH = 7, 8, 10


@pytest.mark.parametrize("T,d,V,nbytes", [(136639, 16, 15522, 34802432), (23318, 16, 150280, 35809536),
                                          (4891, 72, 78308, 22560512), (95810, 64, 25417, 20167424)])
def test_forward_calls_at_earlier_byte_counts(T, d, V, nbytes):
    def loss(have):
        return oapl.lib().oapl_loss_fwd_bwd(X, X, X, X, X, X, X, T, d, V, 1, 1, oapl.OAPL_BF16, 1.0, 1.0, X, X, X, X,
                                            None, None, X, have, None)
    assert loss(nbytes) == ERR_HIP
    assert loss(T * 20) == ERR_WORKSPACE
    assert oapl.lib().oapl_logprob_fwd(X, X, X, T, d, V, oapl.OAPL_BF16, X, X, X, X, nbytes, None) == ERR_HIP
    assert oapl.lib().oapl_sample_tokens(X, X, T, d, V, oapl.OAPL_BF16, 1.0, 1, X, X, X, nbytes, None) == ERR_HIP


@pytest.mark.parametrize("T,d,V,backward", [(72174, 384, 3731, False), (65286, 8, 12834, True), (35944, 16, 13034, True),
                                            (23122, 368, 8894, True), (15303, 416, 34082, False)])
def test_calls_that_fit_the_static_scratch(T, d, V, backward):
    g = X if backward else None
    rc = oapl.lib().oapl_loss_fwd_bwd_noalloc(X, X, X, X, X, X, X, T, d, V, 1, 1, oapl.OAPL_BF16, 1.0, 1.0, X, X, X, X, g, g,
                                              None)
    assert rc == ERR_HIP


# operands at any element: copied where the kernels want them aligned, within byte counts that have always been enough
@pytest.mark.parametrize("T,d,V,forward,one_panel,capped", [(64, 4096, 8192, 70260736, 153344256, 153344256),
                                                            (777, 2048, 3000, 17335552, 48589312, 40688128),
                                                            (8192, 64, 1000, 1541376, 43324672, 5643520),
                                                            (4000, 72, 5003, 2601984, 96377600, 21555968)])
@pytest.mark.parametrize("H,W", [(X + 2, X + 14), (X + 8, X), (X, X + 2)])
def test_operands_that_are_not_aligned(T, d, V, forward, one_panel, capped, H, W):
    L = oapl.lib()
    own = [oapl.workspace_bytes(T, d, V, 0, 1, oapl.OAPL_BF16, False)] + [
        oapl.workspace_bytes(T, d, V, 1, 1, oapl.OAPL_BF16, True, cap) for cap in (None, 384)]
    for sizes in (own, (forward, one_panel, capped)):
        assert L.oapl_logprob_fwd(H, W, X, T, d, V, oapl.OAPL_BF16, X, X, X, X, sizes[0], None) == ERR_HIP
        assert L.oapl_sample_tokens(H, W, T, d, V, oapl.OAPL_BF16, 1.0, 1, X, X, X, sizes[0], None) == ERR_HIP
        for have in sizes[1:]:
            assert L.oapl_loss_fwd_bwd(H, W, X, X, X, X, X, T, d, V, 1, 1, oapl.OAPL_BF16, 1.0, 1.0, X, X, X, X, X, X, X,
                                       have, None) == ERR_HIP
    if sizes[2] <= 64 << 20:
        assert L.oapl_loss_fwd_bwd_noalloc(H, W, X, X, X, X, X, T, d, V, 1, 1, oapl.OAPL_BF16, 1.0, 1.0, X, X, X, X, X, X,
                                           None) == ERR_HIP
