"""Builds the HIP kernels into one shared library, in-tree, for gfx950 only, and the Python entry points on top of it.

    python -m paper_2505_11432_amd.build                    # both
    python -m paper_2505_11432_amd.build --library-only     # the C library: hipcc is all it needs

hipcc cross-compiles without a GPU present.  The library is written next to this file as libmoe_hip.so (public header
include/moe.h); the Python binding reaches it through the extension module _moe_native.so, which needs a host compiler,
Python's headers and torch's, and through ctypes.
"""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from importlib import metadata

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libmoe_hip.so")
CEILINGS_SRC = os.path.join(CSRC, "ceilings", "ceilings.hip")       # measurement aids: a library of their own
CEILINGS_LIB_PATH = os.path.join(HERE, "libmoe_ceilings.so")
NATIVE_SRC = os.path.join(CSRC, "native", "moe_native.cpp")            # Python entry points (host code)
NATIVE_PATH = os.path.join(HERE, "_moe_native.so")
STAMP_PATH = LIB_PATH + ".sha256"      # hash of the sources the library was built from
NATIVE_STAMP_PATH = NATIVE_PATH + ".sha256"
INCLUDE = os.path.join(os.path.dirname(HERE), "include")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
COMMON_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 ALU forms have been unreliable on these boxes: keep the compiler from emitting them
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option", "-Wno-inline-asm",
]


NATIVE_CFLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]
NATIVE_LIBS = ["-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-lmoe_hip", "-Wl,-rpath,$ORIGIN"]


def sources() -> list[str]:
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _hash(words: list[str], files: list[str]) -> str:
    h = hashlib.sha256(" ".join(words).encode())
    for path in sorted(files):
        h.update(os.path.basename(path).encode())
        with open(path, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def source_hash() -> str:
    """SHA-256 over every file the library is compiled from (kernels, internal headers, the public header) and
    the compiler flags."""
    files = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".h"))]
    files += [os.path.join(INCLUDE, f) for f in os.listdir(INCLUDE) if f.endswith(".h")]
    return _hash(COMMON_FLAGS, files + [CEILINGS_SRC])


def native_hash() -> str:
    """The same for the extension module: its source, the C header, the flags, and the interpreter and the torch whose
    objects it reads."""
    try:
        torch_version = metadata.version("torch")
    except metadata.PackageNotFoundError:
        import torch
        torch_version = torch.__version__
    return _hash([CXX, *NATIVE_CFLAGS, *NATIVE_LIBS, str(sysconfig.get_config_var("EXT_SUFFIX")), torch_version],
                 [NATIVE_SRC, os.path.join(INCLUDE, "moe.h")])


def _stamped(stamp_path: str, want: str, *built: str) -> bool:
    if not all(os.path.exists(p) for p in (*built, stamp_path)):
        return False
    with open(stamp_path) as fh:
        return fh.read().strip() == want


def is_current() -> bool:
    """True when the library exists and was built from the sources as they are now."""
    return _stamped(STAMP_PATH, source_hash(), LIB_PATH, CEILINGS_LIB_PATH)


def native_is_current() -> bool:
    """True when the extension module exists and was built from its source for this interpreter and torch."""
    return _stamped(NATIVE_STAMP_PATH, native_hash(), NATIVE_PATH)


def ensure_built() -> str:
    """Build what is not up to date: a library left over from older sources is rebuilt, never used."""
    if not is_current():
        build(verbose=False)
    elif not native_is_current():
        build_native()
    return LIB_PATH


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
    cmd = [HIPCC, *COMMON_FLAGS, "-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_native() -> str:
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(OBJ_DIR, "moe_native.o")
    cmd = [CXX, *NATIVE_CFLAGS, f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem",
           os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem",
           os.path.join(ROCM, "include"), "-isystem", sysconfig.get_paths()["include"], "-c", NATIVE_SRC, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{CXX} failed on {NATIVE_SRC}:\n{res.stderr}")
    if res.stderr.strip():
        sys.stderr.write(res.stderr)
    return obj


def _unstamp(path: str) -> None:
    if os.path.exists(path):
        os.remove(path)                 # no stamp while what is built and the sources may disagree


def _stamp(path: str, value: str) -> None:
    with open(path, "w") as fh:
        fh.write(value + "\n")


def _link(cmd: list[str]) -> None:
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")


def build_library() -> int:
    """The kernels, with hipcc alone; returns the number of sources."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    _unstamp(STAMP_PATH)
    stamp = source_hash()
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as pool:
        ceil_obj = pool.submit(_compile, CEILINGS_SRC)
        objs = list(pool.map(_compile, srcs))
        ceil_obj = ceil_obj.result()
    _link([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", CEILINGS_LIB_PATH, ceil_obj])
    _link([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs])
    _stamp(STAMP_PATH, stamp)
    return len(srcs)


def build_native() -> None:
    """The extension module (needs the library to link against)."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    _unstamp(NATIVE_STAMP_PATH)
    stamp = native_hash()
    obj = _compile_native()
    import torch
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    _link([CXX, "-shared", "-o", NATIVE_PATH, obj, "-L" + torch_lib, "-L" + HERE, *NATIVE_LIBS])
    _stamp(NATIVE_STAMP_PATH, stamp)


def build(verbose: bool = True, native: bool = True) -> str:
    n = build_library()
    if native:
        build_native()
    if verbose:
        print(f"built {LIB_PATH} from {n} sources")
    return LIB_PATH


if __name__ == "__main__":
    build(native="--library-only" not in sys.argv[1:])
