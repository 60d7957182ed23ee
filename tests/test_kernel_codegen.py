"""Static checks of the generated gfx950 code of the matrix-core kernels and of the cross-entropy rows (no GPU needed: hipcc
cross-compiles).

The contraction kernel feeds its pipeline with direct-to-LDS loads written as inline assembly, which the
compiler's wait-count bookkeeping does not see.  If register allocation ever places the reload of a spilled
register inside the contraction loop, the compiler guards it with `s_waitcnt vmcnt(0)`, which also drains
every load of the pipeline: the kernel stays correct and loses 40 % of its speed without any test failing.
These checks read the assembly and fail on that pattern.
"""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2503_01066_amd import build as B


def _device_asm(src):
    cmd = [B._hipcc()] + [f for f in B.FLAGS if f != "-fPIC"] + ["--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


@pytest.fixture(scope="module")
def asm():
    if not (shutil.which(B._hipcc()) or os.path.exists(B._hipcc())):
        pytest.skip("hipcc not found")
    names = {"gemm": "gemm_mfma.hip", "attn": "attn_mfma.hip", "pair": "gemm_pair.hip", "attn64": "attn_mfma_d64.hip", "head": "lmhead.hip",
             "lora": "lora.hip", "generic": "gemm_generic.hip"}
    with ThreadPoolExecutor(max_workers=7) as ex:
        return dict(zip(names, ex.map(_device_asm, names.values())))


def _functions(text, prefix):
    for m in re.finditer(r"^(%s\w*):[^\n]*\n(.*?)^\.Lfunc_end" % prefix, text, re.S | re.M):
        yield m.group(1), m.group(2)


def _blocks(body):
    parts = re.split(r"^(\.LBB\d+_\d+):", body, flags=re.M)
    for i in range(1, len(parts), 2):
        yield parts[i], parts[i + 1]


def _meta(text, name, key):
    # one metadata entry per kernel, "  - .agpr_count: ..." first, keys in alphabetical order
    for entry in re.split(r"^  - \.agpr_count:", text, flags=re.M)[1:]:
        if re.search(r"\.name:\s+%s\n" % re.escape(name), entry):
            return int(re.search(r"\.%s:\s+(\d+)" % key, entry).group(1))
    raise AssertionError("no metadata for " + name)


def test_contraction_loops_hold_no_spill_code_and_no_full_wait(asm):
    seen = 0
    for name, body in _functions(asm["gemm"], "_ZN4alch11k_gemm_mfma"):
        loops = [(lab, txt) for lab, txt in _blocks(body) if txt.count("v_mfma_") >= 16]
        assert loops, name
        for lab, txt in loops:
            assert "scratch_" not in txt, "%s %s: spill code inside a contraction loop" % (name, lab)
            waits = re.findall(r"s_waitcnt ([^\n]*)", txt)
            assert not [w for w in waits if "vmcnt(0)" in w], "%s %s: the loop drains its load pipeline (%s)" % (name, lab, waits)
        seen += 1
    assert seen == 8  # four operand layouts, whole tiles and tiles split along the contraction


def test_attention_kernels_do_not_spill(asm):
    names = [n for n, _ in _functions(asm["attn"], "_ZN4alch")]
    kernels = [n for n in names if "k_attn_" in n]
    assert len(kernels) == 4, kernels  # dQ, dK/dV with and without prefixes, forward
    for n in kernels:
        assert _meta(asm["attn"], n, "vgpr_spill_count") == 0, n
        assert _meta(asm["attn"], n, "private_segment_fixed_size") == 0, n
    for name, body in _functions(asm["attn"], "_ZN4alch19k_attn_bwd_dkv_mfma"):
        for lab, txt in _blocks(body):
            if txt.count("v_mfma_") >= 16:
                assert "scratch_" not in txt, (name, lab)


@pytest.mark.parametrize("prefix,count", [("_ZN4alch11k_gemm_pairI", 4),         # operand layouts
                                          ("_ZN4alch16k_gemm_pair_rowsI", 2)])  # of the right operand, row count on the device
def test_contraction_kernel_of_two_work_groups_keeps_its_registers_and_its_pipeline(asm, prefix, count):
    seen = 0
    for name, body in _functions(asm["pair"], prefix):
        assert _meta(asm["pair"], name, "vgpr_spill_count") == 0 and _meta(asm["pair"], name, "private_segment_fixed_size") == 0, name
        assert _meta(asm["pair"], name, "vgpr_count") <= 256 and _meta(asm["pair"], name, "group_segment_fixed_size") <= 80 * 1024, name
        loops = [(lab, txt) for lab, txt in _blocks(body) if txt.count("v_mfma_") >= 16]
        assert loops, name
        for lab, txt in loops:
            assert "scratch_" not in txt and not re.search(r"s_waitcnt [^\n]*vmcnt\(0\)", txt), (name, lab)
        seen += 1
    assert seen == count


def test_fp32_products_beside_rows_do_not_spill(asm):
    kernels = [n for n, _ in _functions(asm["generic"], "_ZN4alch") if "k_gemm_f32_norm" in n or "k_gemm_f32_gains" in n]
    assert len(kernels) == 3, kernels  # rows of one and of four columns a thread; gain sums
    for n in kernels:
        assert _meta(asm["generic"], n, "vgpr_spill_count") == 0 and _meta(asm["generic"], n, "private_segment_fixed_size") == 0, n


def test_attention_kernels_of_heads_of_64_do_not_spill(asm):
    kernels = [n for n, _ in _functions(asm["attn64"], "_ZN4alch") if "k_attn_" in n or "k_dkv_" in n]
    assert len(kernels) == 6, kernels  # dQ, dK/dV and the sum of its parts with and without prefixes, forward
    for n in kernels:
        assert _meta(asm["attn64"], n, "vgpr_spill_count") == 0 and _meta(asm["attn64"], n, "private_segment_fixed_size") == 0, n
    for name, body in _functions(asm["attn64"], "_ZN4alch19k_attn_bwd_dkv_mfma"):
        # from the first iteration's wait (five loads of a tile may be on their way) to the last matrix instruction
        stream = body[body.index("vmcnt(5)"):body.rindex("v_mfma_")]
        assert stream.count("v_mfma_") >= 48 and "scratch_" not in stream, name
        if "ILi64ELb0E" in name:  # (with prefixes the search for the next sequence reads memory)
            assert not re.search(r"s_waitcnt [^\n]*vmcnt\(0\)", stream), name


def test_cross_entropy_rows_wait_for_no_load_between_request_and_use(asm):
    seen = 0
    for name, body in _functions(asm["head"], "_ZN4alch19k_ce_chunk_bf16_row"):
        assert _meta(asm["head"], name, "vgpr_spill_count") == 0 and _meta(asm["head"], name, "private_segment_fixed_size") == 0, name
        assert _meta(asm["head"], name, "vgpr_count") <= 128, name
        # behind the requests of the next row (direct-to-LDS loads) nothing waits for all of them before the row's own stores
        first = body.index("s_barrier", [m.start() for m in re.finditer(r"offen lds", body)][-1])
        last = body.rindex("buffer_store_dwordx4")
        assert first < last and not re.search(r"s_waitcnt [^\n]*vmcnt\(0\)", body[first:last]), name
        seen += 1
    assert seen == 3  # 4, 8 and 16 chunks of a row


class _Code:
    """Instructions (opcode, operands) of a function and, of each, those that may have run just before it."""
    def __init__(self, body):
        self.ins, labels = [], {}
        for line in body.split("\n"):
            line = line.split(";")[0].strip()
            label = re.match(r"(\.LBB\w+):", line)
            if label:
                labels[label.group(1)] = len(self.ins)
            elif line and not line.startswith(".") and not line.endswith(":"):
                op, _, rest = line.replace("\t", " ", 1).partition(" ")
                self.ins.append((op, rest.strip()))
        self.before = [[i - 1] if i and self.ins[i - 1][0] not in ("s_branch", "s_endpgm") else [] for i in range(len(self.ins))]
        for i, (op, rest) in enumerate(self.ins):
            if op.startswith("s_cbranch") or op == "s_branch":
                self.before[labels[rest.split()[0]]].append(i)

    def loads_into_lds(self):
        return [i for i, (op, rest) in enumerate(self.ins) if op.startswith("buffer_load") and rest.split()[-1] == "lds"]

    def within(self, i, states, found):
        """Whether some path to instruction i meets one that is `found` with fewer than `states` wait states between."""
        for j in self.before[i]:
            op, rest = self.ins[j]
            left = states - (int(rest, 0) + 1 if op == "s_nop" else 1)
            if found(op, rest) or (left > 0 and self.within(j, left, found)):
                return True
        return False


def _scalars(operands):
    out = set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def test_loads_into_lds_wait_for_their_scalars(asm):
    """A buffer load into LDS takes one wait state after a scalar write of m0 and five after a vector instruction's write of
    its descriptor.  The compiler keeps both for loads of its own and looks into no assembly."""
    seen = 0
    for text in asm.values():
        for name, body in _functions(text, "_ZN4alch"):
            code = _Code(body)
            for i in code.loads_into_lds():
                assert not code.within(i, 1, lambda op, rest: op.startswith("s_") and rest.split(",")[0] == "m0"), (name, code.ins[i])
                src = _scalars(code.ins[i][1].partition(",")[2])
                assert not code.within(i, 5, lambda op, rest: op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")) and
                                       _scalars(rest.split(",")[0]) & src), (name, code.ins[i])
                seen += 1
    assert seen > 1000


def test_adapter_rings_are_read_before_they_are_refilled(asm):
    """No read of a wavefront's ring may be on its way when a load into LDS is issued, by a wait that is written there and not
    by one that the compiler places for the products, which it may move."""
    seen = 0
    for name, body in _functions(asm["lora"], "_ZN4alch16k_lora_down_mfma"):
        code = _Code(body)
        assert re.search(r";;#ASMSTART\s+s_waitcnt lgkmcnt\(0\)\s+;;#ASMEND", body), name
        for i in code.loads_into_lds():
            reached, todo = set(), [i]
            while todo:
                for j in code.before[todo.pop()]:
                    op, rest = code.ins[j]
                    assert not op.startswith("ds_read"), (name, code.ins[i])
                    if j not in reached and not (op == "s_waitcnt" and "lgkmcnt(0)" in rest):
                        reached.add(j)
                        todo.append(j)
        seen += 1
    assert seen == 12  # one to four groups of columns, three sizes of work-group


def test_two_contractions_in_one_kernel_keep_their_registers_and_their_pipelines(asm):
    (name, body), = _functions(asm["pair"], "_ZN4alch16k_gemm_two_pairs")
    assert _meta(asm["pair"], name, "vgpr_spill_count") == 0 and _meta(asm["pair"], name, "private_segment_fixed_size") == 0
    assert _meta(asm["pair"], name, "vgpr_count") <= 256 and _meta(asm["pair"], name, "group_segment_fixed_size") <= 80 * 1024
    loops = [txt for lab, txt in _blocks(body) if txt.count("v_mfma_") >= 16]
    # operands with k-major A take steps in pairs, whose waits differ (4 or 8 loads on their way), the others 6
    waits = {w for txt in loops for w in re.findall(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)", txt)}
    assert {"4", "8", "6"} <= waits, waits
    for txt in loops:
        assert "scratch_" not in txt and not re.search(r"s_waitcnt [^\n]*vmcnt\(0\)", txt)
