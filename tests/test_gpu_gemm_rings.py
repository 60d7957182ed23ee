"""The 256x256 contraction kernel where its rings of five stages start, wrap and end: contraction lengths of every remainder by
ten k-tiles, odd numbers of k-tiles and ragged last ones where the contraction is the token index, all operand layouts."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a_k,b_k,lengths", [(True, True, [1024 + 64 * i for i in range(5)]), (True, False, [2752 + 64 * i for i in range(5)]),
                                             (False, True, [1024 + 64 * i for i in range(5)]),
                                             (False, False, [3296 + 32 * i for i in range(10)] + [3301, 3327])])
def test_contraction_lengths(a_k, b_k, lengths):
    # one round of whole tiles, the last column of them ragged: sizes that the estimate gives to this kernel
    import paper_2503_01066_amd as A
    M, N = 4096, 4088
    g = torch.Generator(device="cuda").manual_seed(len(lengths))
    draw = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    for K in lengths:
        a, b = draw(*((M, K) if a_k else (K, M))), draw(*((N, K) if b_k else (K, N)))
        got = A.alch_gemm(M, N, [(a, b, K)], a_k, b_k)
        want = (a if a_k else a.t().contiguous()).float() @ (b.t().contiguous() if b_k else b).float()
        # one rounding to bf16: 2^-9 of the value, on the mean 2^-9 / sqrt(3) of the norm
        err = (got.float() - want).norm() / want.norm()
        assert err < 2 ** -9, (K, float(err))
        assert (got.float() - want).abs().max() <= 2 ** -8 * want.abs().max(), K
