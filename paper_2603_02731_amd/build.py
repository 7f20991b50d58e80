"""Compile the gfx950 kernels and their C ABI into paper_2603_02731_amd/libmxfp4.so, and the native half of the Python
binding into paper_2603_02731_amd/_call_path.*.so (both in-tree)."""
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmxfp4.so")
SOURCES = ["mxfp4_api.hip", "quant_from_fp8.hip", "quant_gather_lists.hip", "quant_from_bf16.hip", "dequant_to_fp8.hip",
           "row_to_col.hip", "row_to_col_segments.hip", "col_small.hip", "row_to_fp8_col.hip", "row_to_fp8_col_requant.hip",
           "row_to_fp8_col_grouped.hip", "stream_copy.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-command-line-argument",
         "-ffp-contract=off",
         # packed-FP32 instructions are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def call_path() -> str:
    """The file of the binding's native half.  It uses PyTorch's C++ interface, which libmxfp4.so does not: its name holds
    the Python and the PyTorch that it is built against, so that another pair does not load it."""
    import torch
    return os.path.join(HERE, f"_call_path.{sysconfig.get_config_var('SOABI')}.torch-{torch.__version__}.so")


def _rocm_include() -> str:
    """Where the HIP headers are: beside the compiler (a path or a name on PATH), under ROCM_PATH or in the usual place."""
    found = shutil.which(HIPCC)
    roots = [os.path.dirname(os.path.dirname(p)) for p in (found, found and os.path.realpath(found)) if p]
    roots += [os.environ.get("ROCM_PATH"), "/opt/rocm"]
    for root in filter(None, roots):
        if os.path.exists(os.path.join(root, "include", "hip", "hip_runtime_api.h")):
            return os.path.join(root, "include")
    raise RuntimeError("no HIP headers beside " + HIPCC)


def _deps(ends):
    out = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(ends)]
    out.append(os.path.join(os.path.dirname(HERE), "include", "mxfp4.h"))
    return out


def _run(cmd, target):
    r = subprocess.run(cmd + ["-o", target + ".tmp"], capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + err)
    if err.strip():
        sys.stderr.write(err + "\n")
    os.replace(target + ".tmp", target)


def _fresh(target, deps):
    return os.path.exists(target) and all(os.path.getmtime(target) >= os.path.getmtime(d) for d in deps)


def build_call_path(force: bool = True) -> str:
    """Host code only: compiled against the headers of the PyTorch that will load it."""
    import torch
    target = call_path()
    if not force and _fresh(target, _deps(".cpp")):
        return target
    t = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", _rocm_include(),
           os.path.join(CSRC, "call_path.cpp"), "-L" + os.path.join(t, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip",
           "-ltorch", "-ltorch_python", "-Wall"]
    _run(cmd, target)
    return target


def build(force: bool = True) -> str:
    if force or not _fresh(LIB, _deps((".hip", ".hpp"))):
        _run([HIPCC] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES], LIB)
    try:
        build_call_path(force)
    except (RuntimeError, OSError) as e:  # the binding works without it, a few microseconds a call slower
        sys.stderr.write(f"the native call path is not built: {e}\n")
        if os.path.exists(call_path()):
            os.remove(call_path())  # of older sources
    return LIB


if __name__ == "__main__":
    print(build(force=True))
