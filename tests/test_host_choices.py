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
    assert ask(("one_pass", 8, last, 8), ("one_pass", 8, last + 64, 8), ("one_pass", 8, 1 << 22, 8)) == [(1,), (0,), (0,)]
