"""Builds libamxfp4.so (HIP kernels + C ABI) for gfx950 with hipcc, and _calls.so, in-tree next to this file.

Run as `python -m paper_2411_09909_amd.build`. hipcc cross-compiles, so no GPU is needed to build.
"""
import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libamxfp4.so")
CALLS = os.path.join(HERE, "_calls.so")
SOURCES = ["gemm_stream.hip", "gemm_stream_glu.hip", "api.hip", "cast.hip", "gemm_bf16.hip", "gemm_fp4.hip", "gemm_e5m2.hip", "gemm_fp8m.hip", "gemm_fp6m.hip", "layer_ops.hip", "peaks.hip", "attention.hip", "attention_64.hip", "attention_decode.hip", "attention_decode_16.hip", "gemm_skinny.hip"]
# packed FP32 VALU ops are switched off on purpose (they have given wrong results on these machines)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-Wall", "-Wno-unused-command-line-argument",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage"]


def spilling_kernels(compiler_output):
    """Kernels whose vector registers did not fit, by the compiler's resource remarks. A build fails on any: the loads in
    flight, the waits and the LDS slots of these kernels are placed by hand for registers, spilled variants are slower, and
    some, of an early form of the stream kernel, gave wrong results whose cause was never found."""
    name, spilling = None, []
    for line in compiler_output.splitlines():
        if "Function Name: " in line:
            name = line.split("Function Name: ")[1].split()[0]
        elif "VGPRs Spill: " in line and int(line.split("VGPRs Spill: ")[1].split()[0]):
            spilling.append(name)
    return spilling


# Kernels that are chosen because so many of their waves fit on a SIMD, with the registers that this leaves each wave.
REGISTERS = {"attention_fused_64_kernel": 96}  # five waves; the kernel of heads of 128, with three, is a sixth to a third slower


def oversized_kernels(compiler_output):
    """Kernels named in REGISTERS that take more vector registers. A build fails on any: nothing else would show it but time."""
    name, oversized = "", []
    for line in compiler_output.splitlines():
        if "Function Name: " in line:
            name = line.split("Function Name: ")[1].split()[0]
        elif "  VGPRs: " in line:
            taken = int(line.split("  VGPRs: ")[1].split()[0])
            oversized += ["%s (it takes %d, %d at most)" % (name, taken, most) for k, most in REGISTERS.items() if k in name and taken > most]
    return oversized


def _diagnostics(compiler_output):
    """The output without the resource remarks, the source lines shown under them and the known harmless warning."""
    kept, remark = [], False
    for line in compiler_output.splitlines():
        remark = "[-Rpass-analysis=kernel-resource-usage]" in line or (remark and re.match(r"\s*\d* \|", line) is not None)
        if not remark and "packed-fp32-ops" not in line and not line.startswith("In file included from "):
            kept.append(line)
    return "\n".join(kept)


def _compile(src):
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = r.stdout + r.stderr
    return src, r.returncode, _diagnostics(out), obj, spilling_kernels(out) + oversized_kernels(out)


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        results = list(ex.map(_compile, SOURCES))
    for src, rc, out, _, spilling in results:
        if out.strip() and verbose:
            print("[%s]\n%s" % (src, out), file=sys.stderr)
        if rc:
            raise RuntimeError("hipcc failed on %s" % src)
        if spilling:
            raise RuntimeError("%s: vector registers spill in %s" % (src, ", ".join(spilling)))
    calls = _start_calls()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + [r[3] for r in results]
    subprocess.check_call(cmd)
    if calls.wait():
        raise RuntimeError("the host compiler failed on calls.cpp")
    return LIB


def _start_calls():
    """Starts the host compiler on the module between torch's tensors and the C ABI (no GPU code in it), for this torch."""
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(cpp_extension.__file__), os.pardir, "lib")
    return subprocess.Popen(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__",
                             "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(),
                             "-DAMX_TORCH_VERSION=\"%s\"" % torch.__version__, os.path.join(CSRC, "calls.cpp"), "-o", CALLS,
                             "-I" + sysconfig.get_path("include")] + ["-isystem" + p for p in cpp_extension.include_paths("cuda")]
                            + ["-L" + os.path.normpath(lib), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])


if __name__ == "__main__":
    print(build())
