"""Builds libalch.so (HIP kernels + C ABI) for gfx950 with hipcc, and _marshal (a Python extension, where that is possible) with g++, in-tree.

Usage: python -m paper_2503_01066_amd.build [--force]
Objects go to _build/ at the repo root; the library to paper_2503_01066_amd/lib/libalch.so.
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

from .binding import torch_build

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "lib", "libalch.so")
MARSHAL = os.path.join(PKG, "_marshal" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))  # (found by the interpreter it is for alone)
SOURCES = ["api.hip", "pack.hip", "gemm_mfma.hip", "gemm_pair.hip", "gemm_narrow.hip", "gemm_generic.hip", "rowops.hip", "attn_generic.hip",
           "attn_mfma.hip", "attn_mfma_d64.hip", "lmhead.hip", "lora.hip", "lora_pass.hip", "dpo.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-inline-asm", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _marshal_stamp():
    return os.path.join(ROOT, "_build", os.path.basename(MARSHAL) + ".torch")


def _marshal_stale():
    """Whether its sources are newer, or it was built with another torch (its date says nothing of that)."""
    if _stale(MARSHAL, [os.path.join(CSRC, "marshal.cpp"), os.path.join(ROOT, "include", "alch.h")]):
        return True
    try:
        with open(_marshal_stamp()) as f:
            return f.read() != torch_build()
    except OSError:
        return True


def _build_marshal(verbose):
    import torch
    t = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-DNDEBUG", '-DALCH_TORCH_BUILD="%s"' % torch_build(),
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I" + os.path.join(t, "include"),
           "-I" + os.path.join(t, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           "-I" + os.path.join(ROOT, "include"), os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL, "-L" + os.path.join(t, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed for marshal.cpp:\n%s" % (cmd[0], r.stderr))
    with open(_marshal_stamp(), "w") as f:
        f.write(torch_build())
    if verbose:
        print("compiled marshal.cpp", flush=True)


def _try_marshal(verbose):
    """The library needs neither this extension nor what it is built with (a host compiler, Python's and torch's headers), and the
    binding does without it: where it cannot be built there is none, and the reason is printed."""
    try:
        _build_marshal(verbose)
    except (RuntimeError, OSError) as e:
        if os.path.exists(MARSHAL):  # (of older sources, or half written)
            os.remove(MARSHAL)
        print("no %s: %s" % (os.path.basename(MARSHAL), e), file=sys.stderr, flush=True)


def build(force=False, verbose=True):
    bdir = os.path.join(ROOT, "_build")
    os.makedirs(bdir, exist_ok=True)
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    headers = [os.path.join(CSRC, h) for h in os.listdir(CSRC) if h.endswith(".h")]
    headers.append(os.path.join(ROOT, "include", "alch.h"))
    jobs = []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(bdir, src.replace(".hip", ".o"))
        if force or _stale(o, [s] + headers):
            jobs.append((s, o))

    def compile_one(job):
        if job is None:
            return _try_marshal(verbose)
        s, o = job
        cmd = [_hipcc()] + FLAGS + ["-c", s, "-o", o]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (s, err))
        if verbose:
            print("compiled", os.path.basename(s), flush=True)

    marshal = force or _marshal_stale()
    with ThreadPoolExecutor(max_workers=min(8, len(jobs) + 1)) as ex:
        list(ex.map(compile_one, ([None] if marshal else []) + jobs))
    objs = [os.path.join(bdir, s.replace(".hip", ".o")) for s in SOURCES]
    if force or jobs or _stale(LIB, objs):
        cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr)
        if verbose:
            print("linked", LIB, flush=True)
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv)
