"""Build libfocused_conv.so in-tree with hipcc for gfx950, and, where PyTorch is installed, the Python extension _native.so beside it.

    python -m paper_2207_10741_amd.build
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys
import tempfile

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
OUT = os.path.join(_HERE, "libfocused_conv.so")
NATIVE = os.path.join(_HERE, "_native.so")          # the Python extension (host code, against PyTorch's C++ interface)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # let the compiler not form packed-fp32 instructions on its own
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]

# sources that hold many kernel instances are compiled as several units (-D<macro>=p), side by side with the others
PARTS = {"fc_conv_mfma.hip": ("FC_MFMA_PART", 6), "fc_conv_wide.hip": ("FC_WIDE_PART", 9)}


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature name and says so: harmless
    noise = ("packed-fp32-ops", "target feature")
    log = "\n".join(ln for ln in res.stdout.splitlines() if not any(n in ln for n in noise))
    if verbose and log.strip():
        print(log, flush=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed (%d): %s\n%s" % (res.returncode, " ".join(cmd), res.stdout))


def _native_command(out):
    """The compile command of the extension, None without PyTorch (the C library needs only ROCm; binding.py makes all calls by itself then)."""
    import sysconfig
    try:
        import torch
    except ImportError:
        return None
    home = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I", os.path.join(ROOT, "include"),
            "-I", os.path.join(home, "include"), "-I", os.path.join(home, "include", "torch", "csrc", "api", "include"),
            "-I", sysconfig.get_paths()["include"], "-I", "/opt/rocm/include", os.path.join(_HERE, "csrc", "fc_python.cpp"), "-o", out,
            "-L", os.path.join(home, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-lamdhip64"]


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    srcs = sorted(glob.glob(os.path.join(_HERE, "csrc", "*.hip")))
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(_HERE, "csrc")]
    jobs = max(1, min(int(os.environ.get("MAX_JOBS", "8")), os.cpu_count() or 1, 8))
    tmp = tempfile.mkdtemp(prefix="fc_build_")
    try:
        units = []      # (object file, compile command); the large units first
        for src in srcs:
            name = os.path.basename(src)
            if name in PARTS:
                macro, parts = PARTS[name]
                for part in range(parts):
                    obj = os.path.join(tmp, "%s.%d.o" % (name, part))
                    units.insert(0, (obj, [hipcc, *HIPCC_FLAGS, *inc, "-D%s=%d" % (macro, part), "-c", src, "-o", obj]))
            else:
                obj = os.path.join(tmp, name + ".o")
                units.append((obj, [hipcc, *HIPCC_FLAGS, *inc, "-c", src, "-o", obj]))
        with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
            native = _native_command(NATIVE + ".tmp")
            for f in [pool.submit(_run, cmd, verbose) for cmd in [cmd for _, cmd in units] + ([native] if native else [])]:
                f.result()
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *[o for o, _ in units], "-o", OUT + ".tmp"], verbose)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    os.replace(OUT + ".tmp", OUT)
    if native:
        os.replace(NATIVE + ".tmp", NATIVE)
    return OUT


if __name__ == "__main__":
    build()
    sys.exit(0)
