"""Builds libmi355conv.so (gfx950 only) from csrc/ with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libmi355conv.so")
MARSHAL = os.path.join(_HERE, "_marshal.so")  # Python extension over LIB (csrc/marshal.cpp), built for one PyTorch and one Python
SOURCES = ["api.cpp", "api_ip.cpp", "kernels_corr.hip", "kernels_corr_patch.hip", "kernels_corr_thin.hip",
           "kernels_small.hip", "kernels_corr_split.hip", "kernels_wgrad_split.hip", "kernels_wgrad.hip", "kernels_bias.hip",
           "kernels_ip.hip", "kernels_pg.hip", "kernels_f64.hip", "kernels_direct.hip", "static_workspace.hip"]
HEADERS = ["internal.h", "device_utils.h", "corr_epilogue.h", "split_bf16.h", "split_f16.h"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 instructions are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix instructions take their accumulators straight from the vector registers: without this
    # the fp64 kernels copy every accumulator to and from the accumulation registers once per k chunk
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-function",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def marshal_target() -> str:
    """What MARSHAL is built for: neither PyTorch's C++ interface nor Python's is the same from one version to the next."""
    import torch
    return f"for torch {torch.__version__} and Python {sys.version_info.major}.{sys.version_info.minor}."


def marshal_fits() -> bool:
    """Whether MARSHAL is there and was built for what is running (it holds the text that marshal_target gave then)."""
    try:
        with open(MARSHAL, "rb") as f:
            return marshal_target().encode() in f.read()
    except OSError:
        return False


def is_stale() -> bool:
    if not os.path.exists(LIB) or not marshal_fits():
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(MARSHAL))
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS + ["marshal.cpp"]] + [
        os.path.join(_ROOT, "include", h) for h in ("mi355conv.h", "mi355ip.h", "mi355pg.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def _torch_dir() -> str:
    import torch
    return os.path.dirname(torch.__file__)


def _compile_marshal(obj_dir: str) -> str:
    """Host code only: the extension calls the C entry points of LIB."""
    import sysconfig

    torch_include = os.path.join(_torch_dir(), "include")
    obj = os.path.join(obj_dir, "marshal.o")
    rocm = os.path.dirname(os.path.dirname(_hipcc())) if os.path.isabs(_hipcc()) else "/opt/rocm"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", "-w",
           f'-DMARSHAL_TARGET="{marshal_target()}"',
           "-I", os.path.join(_ROOT, "include"), "-isystem", torch_include,
           "-isystem", os.path.join(torch_include, "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
           "-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj]
    res = subprocess.run(cmd, cwd=CSRC, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + " ".join(cmd) + "\n" + res.stdout + res.stderr)
    return obj


def _link_marshal(obj: str) -> None:
    torch_lib = os.path.join(_torch_dir(), "lib")
    cmd = ["g++", "-shared", "-o", MARSHAL, obj, "-L", _HERE, "-l:libmi355conv.so", "-Wl,-rpath,$ORIGIN",
           "-L", torch_lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, cwd=_HERE, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ link failed:\n" + " ".join(cmd) + "\n" + res.stdout + res.stderr)


def build_marshal() -> None:
    """The extension alone, over the library that is there."""
    obj_dir = os.path.join(_HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    _link_marshal(_compile_marshal(obj_dir))


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every kernel for gfx950 (one hipcc process per source file, side by side) and link the
    C-ABI library next to this file."""
    if not force and not is_stale():
        return LIB
    from concurrent.futures import ThreadPoolExecutor

    obj_dir = os.path.join(_HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    include = ["-I", os.path.join(_ROOT, "include"), "-I", CSRC]

    def compile_one(src: str) -> str:
        obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
        cmd = [_hipcc(), *flags, *include, "-c", os.path.join(CSRC, src), "-o", obj]
        res = subprocess.run(cmd, cwd=CSRC, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + res.stdout + res.stderr)
        if verbose:
            print(res.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        marshal = pool.submit(_compile_marshal, obj_dir)
        objs = list(pool.map(compile_one, SOURCES))
        marshal_obj = marshal.result()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    res = subprocess.run(cmd, cwd=CSRC, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc link failed:\n" + " ".join(cmd) + "\n" + res.stdout + res.stderr)
    _link_marshal(marshal_obj)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
