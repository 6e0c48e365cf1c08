"""Builds libitq3s.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libitq3s.so")
SOURCES = ["itq3s_api.hip", "itq3s_quantize.hip", "itq3s_dequantize.hip", "itq3s_rotate.hip", "itq3s_gemv.hip", "itq3s_rows.hip", "itq3s_gemm.hip", "itq3s_mx.hip", "itq3s_gemm_ws.hip", "itq3s_probe.hip", "itq3s_ablation.hip"]
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # every floating-point operation rounds on its own (the quantizer is specified bit for bit);
    # fused multiply-adds are written explicitly where wanted
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
]
# the first kernel arguments arrive in scalar registers instead of through a fetch from memory that
# everything else waits for (a rotation launch plus the streaming launch behind it: 0.25 us less)
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
# where the way to the first load is not what counts it only costs: quantizer 0.12 us of every call (4.7 -> 4.8)
NO_PRELOAD = ("itq3s_quantize.hip",)


def flags(source):
    return FLAGS + ([] if os.path.basename(source) in NO_PRELOAD else PRELOAD)


def build_lib(force=True, verbose=False):
    """Compile every kernel source and link the shared library.  Returns its path."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    deps = srcs + [os.path.join(CSRC, h) for h in os.listdir(CSRC) if h.endswith(".h")] + [os.path.join(HERE, "..", "include", h) for h in ("itq3s.h", "itq3s_bench.h")]
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    objs = []
    procs = []
    for s in srcs:
        o = s[:-4] + ".o"
        objs.append(o)
        cmd = ["hipcc", *flags(s), "-c", s, "-o", o]
        if verbose:
            print(" ".join(cmd))
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            raise RuntimeError("hipcc failed: %s\n%s" % (" ".join(cmd), out))
        if verbose and out:
            print(out)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build_lib(verbose=True))
