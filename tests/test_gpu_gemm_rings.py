"""The 256x256 contraction kernel where its rings of five stages start, wrap and end: contraction lengths of every remainder by
ten k-tiles, odd numbers of k-tiles and ragged last ones where the contraction is the token index, all operand layouts.  Shorter
token-major contractions of the same size run on the 128x256 kernel (test_host_choices.py holds both lists to that)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

M, N = 4096, 4088  # one round of whole tiles, the last column of them ragged
CASES = [(True, True, [1024 + 64 * i for i in range(5)]), (True, False, [2752 + 64 * i for i in range(5)]),
         (False, True, [1024 + 64 * i for i in range(5)]), (False, False, [3520 + 32 * i for i in range(10)] + [3525, 3551, 3809])]
OTHER_KERNEL = (False, False, [3296 + 32 * i for i in range(6)] + [3301, 3327])


@pytest.mark.parametrize("a_k,b_k,lengths", CASES + [OTHER_KERNEL])
def test_contraction_lengths(a_k, b_k, lengths):
    import paper_2503_01066_amd as A
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
