"""Which kernel a call takes, as the host decides it: asked of the library by a small program (tests/host_choices.cpp), without a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2503_01066_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if not (shutil.which(B._hipcc()) or os.path.exists(B._hipcc())):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "choices")
    cmd = [B._hipcc()] + [f for f in B.FLAGS if f != "-fPIC"] + ["--cuda-host-only", "-x", "hip", os.path.join(HERE, "host_choices.cpp"),
                                                                 "-x", "none", B.LIB, "-rdynamic", "-Wl,-rpath," + os.path.dirname(B.LIB), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def ask(*questions):
        r = subprocess.run([exe], input="\n".join(" ".join(str(int(x) if isinstance(x, bool) else x) for x in q) for q in questions),
                           capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        out = [line.split() for line in r.stdout.splitlines()]
        assert len(out) == len(questions)
        return [tuple(int(x) for x in line) for line in out]
    return ask


def test_contraction_length_on_the_device_needs_token_major_operands(ask):
    """The kernels take a k-major operand 64 k at a time, and only the host can see that a length is a multiple of that."""
    forms = [(a, b) for a in (False, True) for b in (False, True)]
    known = ask(*[("supported", 512, 512, 256, a, b, False) for a, b in forms])
    assert known == [(1,)] * 4
    dev = ask(*[("supported", 512, 512, 256, a, b, True) for a, b in forms])
    assert dev == [(1,), (0,), (0,), (0,)]


def test_adapter_pass_takes_no_rows_that_its_launch_refuses(ask):
    """[dG | dU] rows of 2^22 elements and more: beyond the offsets of the pass (128 rows below 2^29 elements), so the layer takes the
    separate kernels; a layer that found this out at the launch had failed half way."""
    last = (1 << 21) - 64  # [dG | dU] has two of them to a row
    assert ask(*[("one_pass", 8, 64, ffn, 8) for ffn in (last, last + 64, 1 << 22)]) == [(1,), (0,), (0,)]


# ---- the GPU tests that are about one kernel reach it (256 compute units)
def test_ring_lengths_run_on_the_kernel_with_the_rings(ask):
    from test_gpu_gemm_rings import CASES, M, N, OTHER_KERNEL
    for a_k, b_k, lengths in CASES:
        assert ask(*[("kernel", M, N, K, a_k, b_k) for K in lengths]) == [(0,)] * len(lengths), (a_k, b_k)
        step = 64 if a_k or b_k else 32
        assert {K // step % (320 // step) for K in lengths} == set(range(320 // step)), (a_k, b_k)  # where the rings end
    a_k, b_k, lengths = OTHER_KERNEL
    assert ask(*[("kernel", M, N, K, a_k, b_k) for K in lengths]) == [(1,)] * len(lengths)


def test_long_kept_rows_run_on_the_kernel_with_the_rings(ask):
    from test_gpu_kept_rows_products import LONG, LONG_T
    hidden, n_q, n_kv, head_dim, ffn = LONG[:5]
    half = LONG_T // 2  # (the choice is that for half of the tokens)
    assert ask(("kernel", 2 * ffn, hidden, half, False, False)) == [(0,)]


def test_rows_beside_products_share_their_launch(ask):
    from test_gpu_rows_beside_products import APART, BESIDE, QKV
    beside = lambda cases: ask(*[("rows_beside", hidden, ffn, T, QKV) for hidden, ffn, T in cases])
    assert beside(BESIDE) == [(1, 1)] * len(BESIDE)
    assert beside(APART) == [(0, 0)] * len(APART)


def test_pairs_of_batches_differ_in_the_pass_and_not_in_the_parts_of_t2(ask):
    from test_gpu_lora_pass import BITS, BITS_SHAPE
    hidden, ffn = BITS_SHAPE[0], BITS_SHAPE[4]
    for rank, in_one, apart in BITS:
        assert ask(("one_pass", in_one, hidden, ffn, rank), ("one_pass", apart, hidden, ffn, rank)) == [(1,), (0,)]
        for problems in (1, 2):  # of d by itself, of gate and up
            p = ask(("t_parts", in_one, problems), ("t_parts", apart, problems))
            assert p[0] == p[1], (in_one, apart, problems)
    assert {ask(("t_parts", b[1], 2))[0] for b in BITS} == {(16,), (8,), (4,)}


def test_short_sequences_lie_beside_cut_key_blocks(ask):
    from test_gpu_attention_short import CUT
    for heads, lens in CUT:
        (up_to, parts, both), = ask(("attention", 64, heads, 1, 1024, False, len(lens), *lens))
        assert up_to == 8 and parts > 1 and not both, (heads, lens)


def test_kept_rows_are_products_that_the_matrix_core_kernels_take(ask):
    """The products of a masked layer by their largest operands, beside what the kernels say of each."""
    for T, H, F, QD in [(256, 64, 1 << 20, 256), (256, 64, (1 << 20) + 64, 256), (256, 1024, (1 << 20) - 64, 256), (256, 1024, 1 << 20, 256),
                        (140000, 8192, 64, 256), (70000, 64, 64, 1 << 14), (8192, 8192, 28672, 8192), (300, 8192, 131072, 256), (300, 96, 256, 64)]:
        data = ask(("supported", T, F, H, True, False, False), ("supported", T, H, F, True, False, False), ("supported", T, QD, H, True, False, False),
                   ("supported", 2 * F, H, T, False, False, True), ("supported", H, F, T, False, False, True), ("supported", H, QD, T, False, False, True))
        wide = 2 * F <= 1 << 21 and T * 2 * F * 2 < 1 << 31  # ([dG | dU] as the left operand of dH2)
        assert ask(("kept_rows", T, H, F, QD)) == [(all(d == (1,) for d in data) and wide,)], (T, H, F, QD, data)


BIG, PAIR, NARROW64, NARROW128 = range(4)


def _data_gradients(hidden, ffn, qd, V, rows, several):
    """dHf, dAct, dH2, dO of so many kept rows."""
    return [("rows", rows, n, k, swiglu, several) for n, k, swiglu in ((hidden, V, False), (ffn, hidden, True), (hidden, 2 * ffn, False), (qd, hidden, False))]


def test_few_kept_rows_of_several_layers_run_in_narrow_tiles(ask):
    from test_gpu_narrow_rows import CASES, QD
    seen = set()
    for hidden, ffn, V, T, kept, wstd in CASES:
        kernels = [k for k, _ in ask(*_data_gradients(hidden, ffn, QD, V, kept, True))]
        assert set(kernels) <= {NARROW64, NARROW128}, (hidden, ffn, kept, kernels)
        seen |= set(enumerate(kernels))
    assert seen == {(product, k) for product in range(4) for k in (NARROW64, NARROW128)} - {(3, NARROW128)}  # (dO: 256 columns)


def test_rows_compared_by_their_bits_run_on_different_kernels(ask):
    from test_gpu_narrow_rows import BITS, BITS_SHAPE, BITS_V, QD
    hidden, ffn = BITS_SHAPE[0], BITS_SHAPE[4]
    seen = set()
    for few, many in BITS:
        a, b = [[k for k, _ in ask(*_data_gradients(hidden, ffn, QD, BITS_V, rows, True))[:3]] for rows in (few, many)]
        assert set(a) <= {NARROW64, NARROW128} | ({PAIR, BIG} if few > 1024 else set()) and set(b) <= {BIG, PAIR}, (few, many, a, b)
        assert a[0] in (NARROW64, NARROW128)
        seen |= set(enumerate(a))
    assert {(product, k) for product in range(3) for k in (NARROW64, NARROW128)} <= seen


def test_head_gradients_of_few_kept_rows_are_cut(ask):
    from test_gpu_kept_rows_heads import KEPT, SIZES
    for hidden, V in SIZES:
        assert all(kernel == PAIR and parts > 1 for kernel, parts in ask(*[("rows", kept, hidden, V, False, False) for kept in KEPT])), (hidden, V)


def test_short_batches_run_both_attention_gradients_as_one(ask):
    from test_gpu_attention_both import APART, BITS, BITS_FFN, FFN, HEADS, LENS, OTHERS, WIDE_FFN, WIDE_LENS
    asked = lambda h, lens, ffn, several: ("attention", h[2], h[0], h[1], ffn, several, len(lens), *lens)
    for h in HEADS:
        for lens, (_, parts, both) in zip(LENS, ask(*[asked(h, lens, FFN, False) for lens in LENS])):
            assert both == ((h, lens) not in APART) and (parts > 1) == (h == (32, 1, 64)), (h, lens)
    for h in HEADS[:2]:
        assert all(both and parts > 1 for _, parts, both in ask(*[asked(h, lens, WIDE_FFN, False) for lens in WIDE_LENS])), h
    assert ask(*[asked(h, lens, BITS_FFN, True) for h, lens in BITS]) == [(0, 1, 1)] * len(BITS)
    assert ask(*[asked(h, lens + OTHERS, BITS_FFN, True) for h, lens in BITS]) == [(0, 1, 0)] * len(BITS)


def test_masked_adapter_layers_run_on_their_kept_rows(ask):
    from test_gpu_lora_kept_rows import ALL_ROWS, CASES
    for T, rank, hidden, ffn, frozen, accumulate in CASES:
        on_kept_rows = all(a == (1,) for a in ask(("one_pass", T, hidden, ffn, rank), ("adapters_pay", T, hidden, ffn), ("kept_rows", T, hidden, ffn, 256)))
        assert on_kept_rows == (T not in ALL_ROWS), T
