"""Build libsw_decode.so (hand-written HIP for gfx950) and sw_native (its Python caller) in-tree.

    python -m paper_2311_18677_amd.build

Compiles every time it is called; the tests, smoke() and bench.py only load
what is already built.
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsw_decode.so")
# the Python side of a call (csrc/sw_python.cpp); named for the interpreter whose object layouts it is
# compiled against, so that no other one imports it
NATIVE = os.path.join(HERE, "sw_native" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["sw_api.hip", "sw_partial_valu.hip", "sw_decode_split.hip", "sw_combine.hip", "sw_lens.hip", "sw_prefill_mfma.hip", "sw_kv_handoff.hip", "sw_prefill_split.hip", "sw_prefill_halves.hip", "sw_calibrate.hip", "sw_kv_store.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # leading scalar kernel arguments arrive in registers with the wave (the decode kernel's
    # length scan starts from them); kernels whose first argument is a struct are unaffected
    "-mllvm", "-amdgpu-kernarg-preload-count=8",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src):
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_native():
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
           "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "sw_python.cpp"), "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("%s failed on sw_python.cpp:\n%s" % (cmd[0], res.stderr))
    os.replace(tmp, NATIVE)
    unnamed = os.path.join(HERE, "sw_native.so")
    if os.path.exists(unnamed) and unnamed != NATIVE:          # of a build before, which any interpreter would take
        os.unlink(unnamed)


def build(verbose=False):
    os.makedirs(OBJ_DIR, exist_ok=True)
    _build_native()
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    # every symbol must resolve: load the result once, in a process of its own
    chk = subprocess.run([sys.executable, "-c", "import ctypes, sys; ctypes.CDLL(sys.argv[1], mode=2)", tmp],
                         capture_output=True, text=True)
    if chk.returncode != 0:
        os.unlink(tmp)
        raise RuntimeError("the built library does not load:\n" + chk.stderr)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
