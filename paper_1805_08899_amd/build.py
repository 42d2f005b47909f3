"""Builds libechoattn.so from csrc/*.hip for gfx950 with hipcc, and _py_calls.so, the Python binding's argument
marshalling, from csrc/py_calls.cpp with g++ (in-tree; the latter needs PyTorch's headers and is left out without them).

    python -m paper_1805_08899_amd.build [--sanitize] [extra hipcc flags]

Objects go to paper_1805_08899_amd/_build/, the library next to this file.
hipcc cross-compiles without a GPU present.

--sanitize builds a second library, _build/libechoattn_san.so, whose HOST code carries AddressSanitizer and
UndefinedBehaviorSanitizer instrumentation (the device code is built as usual: sanitizers for device code are not
available here).  It is for the host-side walk through the argument checks in tests/host/, never for the GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libechoattn.so")
PY_CALLS = os.path.join(HERE, "_py_calls.so")

# Packed fp32 VALU forms are switched off for all device code.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-parameter",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


SAN_LIB = os.path.join(OBJ, "libechoattn_san.so")
# each -fsanitize= directly behind -Xarch_host, so that only the host pass sees it
SAN_COMPILE = ["-g", "-fno-omit-frame-pointer", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
               "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=undefined"]
SAN_LINK = ["-fsanitize=address,undefined", "-fno-gpu-sanitize", "-shared-libsan"]


def _compile(src: str, extra, suffix: str = "") -> str:
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + suffix + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, *extra, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "is not a recognized feature for this target" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
    if msgs.strip():
        print(msgs, file=sys.stderr)
    return obj


def build_py_calls() -> None:
    """_py_calls.so: host code only, against the headers of the PyTorch that will import it."""
    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        return
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]
    lib_dirs = cpp_extension.library_paths()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(a for d in inc for a in ("-isystem", d)),
           os.path.join(CSRC, "py_calls.cpp"), "-o", PY_CALLS, *("-L" + d for d in lib_dirs),
           "-lc10", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for py_calls.cpp:\n" + r.stdout + r.stderr)
    if (r.stdout + r.stderr).strip():
        print(r.stdout + r.stderr, file=sys.stderr)


def build_library(extra_flags=(), verbose=True, sanitize=False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    flags = list(extra_flags) + (SAN_COMPILE if sanitize else [])
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        py_calls = None if sanitize else ex.submit(build_py_calls)
        objs = list(ex.map(lambda s: _compile(s, flags, "_san" if sanitize else ""), srcs))
        if py_calls:
            py_calls.result()
    out = SAN_LIB if sanitize else LIB
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *(SAN_LINK if sanitize else []), "-o", out, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    if verbose:
        print(f"built {out} from {len(srcs)} sources")
    return out


if __name__ == "__main__":
    args = sys.argv[1:]
    san = "--sanitize" in args
    build_library([a for a in args if a != "--sanitize"], sanitize=san)
