"""Build the C-ABI library (librbgp.so) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "librbgp.so")
# the binding's calls without ctypes (csrc/rbgp_call.c), for this interpreter only: another one's objects are laid out otherwise
CALL = os.path.join(_HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["rbgp_mfma_reg_bf16_wide.hip", "rbgp_mfma_reg_bf16.hip", "rbgp_mfma_reg_bf16_lean.hip", "rbgp_mfma_reg.hip", "rbgp_host.cpp",
           "rbgp_device.hip", "rbgp_mfma_reg_dual.hip", "rbgp_mfma_reg_split.hip",
           "rbgp_mfma_reg_bf16_shared.hip", "rbgp_mfma_reg_rows.hip", "rbgp_mfma_reg_narrow.hip", "rbgp_conv_tile.hip", "rbgp_sddmm.hip", "rbgp_sddmm_lines.hip", "rbgp_mfma_tile.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=default",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    """Compile every source and link librbgp.so (always recompiles).  extra: more hipcc flags."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc, *FLAGS, *(extra or []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + out)
        if verbose and out.strip():
            print(out)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.check_call(cmd)
    build_call()
    return LIB


def build_call(out: str = CALL) -> bool:
    """Compile the binding's calls without ctypes.  The binding does without them (see binding.py), so where there is no C compiler or
    Python's headers are not installed that is said and no older file left in their place."""
    for name in os.listdir(os.path.dirname(out)):
        if name.startswith("_call.") and name.endswith(".so"):
            os.remove(os.path.join(os.path.dirname(out), name))
    try:
        subprocess.check_call([os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"],
                               "-o", out, os.path.join(CSRC, "rbgp_call.c")])
    except (OSError, subprocess.CalledProcessError) as e:
        print(f"{os.path.basename(out)} is not built ({e}): the binding's calls go through ctypes", file=sys.stderr)
        return False
    return True


def build_sanitized() -> str:
    """The same library with its HOST code under AddressSanitizer and UndefinedBehaviorSanitizer (device code is
    compiled as usual): librbgp_asan.so, for the CPU tests of the host logic -- sampler, index tables, layouts,
    transposes -- which run it in a child process with the sanitizer runtime preloaded (tests/test_host_sanitizers.py)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host",
           "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer", "-g"]
    flags = [f if f != "-O3" else "-O1" for f in FLAGS]
    lib = os.path.join(_HERE, "librbgp_asan.so")
    objs, procs = [], []
    for src in SOURCES:
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".asan.o")
        cmd = [hipcc, *flags, *san, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for cmd, p in procs:
        out, _ = p.communicate()
        if p.returncode:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + out)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fsanitize=address", "-fsanitize=undefined",
                           "-shared-libsan", "-o", lib, *objs])
    return lib


def sanitizer_runtime() -> str:
    """The AddressSanitizer runtime that librbgp_asan.so needs preloaded (clang's, from the ROCm toolchain)."""
    import glob
    found = sorted(glob.glob("/opt/rocm/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so"))
    if not found:
        raise RuntimeError("no libclang_rt.asan-x86_64.so under /opt/rocm/llvm")
    return found[-1]


if __name__ == "__main__":
    print(build_sanitized() if "sanitized" in sys.argv else build(verbose="-v" in sys.argv))
