"""Compiles the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU), and the
compiled part of the Python binding, which is host code only."""
from __future__ import annotations

import json
import os
import re
import shutil
import subprocess
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "pcgrl_api.hip")
DEPS = [SRC, os.path.join(HERE, "csrc", "pcgrl_kernels.hip.h"), os.path.join(HERE, "csrc", "pcgrl_index.h"),
        os.path.join(HERE, "csrc", "pcgrl_relay.h"), os.path.join(HERE, "csrc", "pcgrl_spans.h"),
        os.path.join(HERE, "csrc", "pcgrl_split.h"),
        os.path.join(os.path.dirname(HERE), "include", "pcgrl.h")]
LIB_DIR = os.path.join(HERE, "_lib")
LIB = os.path.join(LIB_DIR, "libpcgrl.so")
PY_SRC = os.path.join(HERE, "csrc", "pcgrl_py.cpp")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep hipcc from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the reward is a sum of float32 products in a fixed order: no fused multiply-adds
    "-ffp-contract=off",
    # leading scalar kernel arguments (up to 8 of them, 14 dwords) are preloaded into scalar
    # registers at wavefront launch; the step kernel is written for that
    "-mllvm", "-amdgpu-kernarg-preload-count=8",
]


def py_lib() -> str:
    """Path of the binding's compiled part.  Unlike the library it is good for one interpreter and one
    torch only (it reads torch's C++ objects), so its name carries both, and after a change of either
    it counts as not built."""
    import torch
    return os.path.join(LIB_DIR, "pcgrl_py.%s.torch-%s.so" % (sysconfig.get_config_var("SOABI"), torch.__version__))


def is_stale() -> bool:
    newest = lambda files: max(os.path.getmtime(f) for f in files)
    return (not os.path.exists(LIB) or os.path.getmtime(LIB) < newest(DEPS) or not os.path.exists(py_lib()) or
            os.path.getmtime(py_lib()) < newest([PY_SRC, DEPS[-1]]))


SCAN_REPORT = os.path.join(LIB_DIR, "libpcgrl.scan.json")
_SHIFT64 = re.compile(r"\s*(v_lshlrev_b64|v_lshrrev_b64|v_ashrrev_i64)\s+v\[\d+:\d+\],\s*(\S+),")


def scan_shift_amounts(asm_text: str):
    """Looks through the device assembly of this library for 64-bit vector shifts whose shift
    amount sits in the highest vector register of the kernel's allocation (registers are handed
    out in blocks of eight).  On the MI355X boxes this library is measured on such a shift gives
    wrong results in about a tenth of the lanes once several wavefronts share a SIMD (found with
    the 64x64 maze kernel for wide windows, confirmed with a twenty-line probe kernel: the same
    shift with its amount four registers lower is always right).  The compiler works round this
    for another GPU generation only, so the build checks for it.
    Returns (number of kernels, [(kernel, allocation, instruction), ...])."""
    body, alloc, cur, kern = {}, {}, None, None
    for line in asm_text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = m.group(1)
            body[cur] = []
            continue
        m = re.match(r"\s*\.amdhsa_kernel (\w+)", line)
        if m:
            kern = m.group(1)
            continue
        m = re.match(r"\s*\.amdhsa_next_free_vgpr (\d+)", line)
        if m and kern:
            alloc[kern] = int(m.group(1))
            continue
        if cur:
            body[cur].append(line)
    found = []
    for k, n in alloc.items():
        top = (n + 7) // 8 * 8 - 1
        for line in body.get(k, []):
            m = _SHIFT64.match(line)
            if m and m.group(2) == f"v{top}":
                found.append((k, top + 1, line.strip()))
    return len(alloc), found


def kernel_resources(asm_text: str):
    """What each kernel of the device assembly takes: vector registers, bytes of scratch memory and of LDS (without
    what a launch adds), and the vector loads from memory that stand in its code.  Returns
    {kernel: {"vgprs", "scratch", "lds", "loads"}}."""
    fields = {"amdhsa_next_free_vgpr": "vgprs", "amdhsa_private_segment_fixed_size": "scratch", "amdhsa_group_segment_fixed_size": "lds"}
    out, loads, cur, kern = {}, {}, None, None
    for line in asm_text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = m.group(1)
            loads[cur] = 0
        elif cur and re.match(r"\s+(global|flat|scratch|buffer)_load_", line):
            loads[cur] += 1
        m = re.match(r"\s*\.(amdhsa_\w+)\s+(\w+)", line)
        if m and m.group(1) == "amdhsa_kernel":
            kern = m.group(2)
            out[kern] = {"loads": loads.get(kern, 0)}
        elif m and m.group(1) in fields:
            out[kern][fields[m.group(1)]] = int(m.group(2))
    return out


def build(force: bool = True, verbose: bool = False) -> str:
    """Runs hipcc; with force=False only when the library is missing or older than its sources.
    The device assembly the compiler leaves behind is checked by scan_shift_amounts(); a finding
    fails the build (the kernel it names then needs one more register block, see step_kernel)."""
    if force or is_stale():
        os.makedirs(LIB_DIR, exist_ok=True)
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        tmp = tempfile.mkdtemp(prefix="pcgrl_build_")
        try:
            out = os.path.join(tmp, "libpcgrl.so")
            cmd = [hipcc] + HIPCC_FLAGS + ["-save-temps", "-o", out, SRC]
            if verbose:
                print(" ".join(cmd), flush=True)
            res = subprocess.run(cmd, cwd=tmp, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            if res.returncode != 0:
                raise RuntimeError("hipcc failed:\n" + res.stdout)
            asm = [f for f in os.listdir(tmp) if f.endswith("gfx950.s")]
            if len(asm) != 1:
                raise RuntimeError("device assembly not found among the compiler's temporaries: %s" % os.listdir(tmp))
            with open(os.path.join(tmp, asm[0])) as f:
                text = f.read()
            n_kernels, found = scan_shift_amounts(text)
            with open(SCAN_REPORT, "w") as f:
                json.dump({"kernels": n_kernels, "findings": found, "resources": kernel_resources(text)}, f)
            if found:
                raise RuntimeError("64-bit shifts with their amount in the highest allocated vector register:\n" +
                                   "\n".join("  %s (allocation %d): %s" % t for t in found))
            shutil.move(out, LIB)
        finally:
            shutil.rmtree(tmp, ignore_errors=True)
        build_py(verbose)
    return LIB


def build_py(verbose: bool = False) -> str:
    """Compiles csrc/pcgrl_py.cpp against the installed torch and the library in-tree."""
    import torch
    troot = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = tempfile.mkdtemp(prefix="pcgrl_build_")
    try:
        out = os.path.join(tmp, "pcgrl_py.so")
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
               "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
               "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
               "-I" + os.path.join(troot, "include"),
               "-I" + os.path.join(troot, "include", "torch", "csrc", "api", "include"),
               "-I" + os.path.join(rocm, "include"), "-I" + sysconfig.get_paths()["include"],
               PY_SRC, "-o", out, "-L" + LIB_DIR, "-l:libpcgrl.so", "-L" + os.path.join(troot, "lib"),
               "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if res.returncode != 0:
            raise RuntimeError("the Python binding's compiled part failed to build:\n" + res.stdout)
        shutil.move(out, py_lib())
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return py_lib()


if __name__ == "__main__":
    print(build(verbose=True))
