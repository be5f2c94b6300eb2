"""Builds libsparseffn.so (HIP, gfx950) in-tree with hipcc."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsparseffn.so")
SOURCES = ["api.hip", "prune24.hip", "vnm.hip", "vnm_general.hip", "gemm_v2.hip", "gemm_v2_row.hip", "forward_x.hip", "gemm_v2_fp8.hip", "step_mix_bf16.hip", "step_mix_wide.hip", "step_mix_fp8.hip", "step_mix_fp8_wide.hip", "prologue.hip", "prologue_fp8.hip", "gemm_wgrad.hip", "gemm_wgrad_wide.hip", "gemm_gather.hip", "gemm_vnm8.hip", "router.hip", "router_mix.hip", "dense_ref.hip", "noalloc.hip", "fp8.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
         # accumulators in VGPRs: where one wavefront has a SIMD to itself the compiler takes AGPRs and moves the 16 x 16 instructions' sums between the two in the loop
         "-mllvm", "-amdgpu-mfma-vgpr-form"]


def build(verbose=False, extra_flags=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed: %s\n%s" % (" ".join(cmd), out))
        if verbose and out.strip():
            print(out)
    cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed: %s\n%s" % (" ".join(cmd), r.stdout))
    return LIB


def build_host_sanitized(driver_cpp, exe):
    """The library's sources plus a host-side driver as one executable whose HOST code runs under AddressSanitizer and
    UndefinedBehaviorSanitizer (device code is compiled as usual and never launched by the driver).  Returns the executable."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=undefined", "-g"]
    outdir = os.path.join(HERE, "_build", "san")
    os.makedirs(outdir, exist_ok=True)
    procs, objs = [], []
    for src in SOURCES + [driver_cpp]:
        path = src if os.path.isabs(src) else os.path.join(CSRC, src)
        obj = os.path.join(outdir, os.path.basename(path).rsplit(".", 1)[0] + ".o")
        objs.append(obj)
        flags = FLAGS if path.endswith(".hip") else ["-O1", "-std=c++17", "-fPIC"]
        cmd = [hipcc, *flags, *san, "-c", path, "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for cmd, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError("hipcc failed: %s\n%s" % (" ".join(cmd), out))
    cmd = [hipcc, "--offload-arch=gfx950", "-fsanitize=address,undefined", "-fno-gpu-sanitize", "-o", exe, *objs]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed: %s\n%s" % (" ".join(cmd), r.stdout))
    return exe


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
