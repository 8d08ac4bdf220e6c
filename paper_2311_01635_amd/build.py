"""Build librtp.so (HIP kernels for gfx950 + the host scheduler) in-tree with hipcc."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librtp.so")
# (the files that take longest to compile first)
SOURCES = ["rtp_gemm_pp_nt.hip", "rtp_gemm_pp_nn.hip", "rtp_gemm_pp_tn.hip",
           "rtp_gemm_pp_nt_f16.hip", "rtp_gemm_pp_nn_f16.hip", "rtp_gemm_pp_tn_f16.hip",
           "rtp_gemm_bf16.hip", "rtp_gemm_pp_nn_tn.hip", "rtp_gemm_pp_nn_tn_f16.hip",
           "rtp_gemm_duo_nt.hip", "rtp_gemm_duo_nn_tn.hip", "rtp_gemm_duo_nt_f16.hip", "rtp_gemm_duo_nn_tn_f16.hip",
           "rtp_gemm_pp.hip", "rtp_misc_kernels.hip", "rtp_host.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops off: the compiler must not form packed fp32 arithmetic from scalar code
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-x", "hip"]


def _newer(dst, srcs):
    return os.path.exists(dst) and all(os.path.getmtime(dst) >= os.path.getmtime(s) for s in srcs)


def build(force: bool = True, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    kernel_headers = [os.path.join(CSRC, h) for h in ("rtp_kernels.h", "rtp_ride.h", "rtp_gemm_epilogue.h", "rtp_gemm_pp.h", "rtp_gemm_small.h", "rtp_gemm_duo.h")]
    host_headers = [os.path.join(CSRC, "rtp_kernels.h"), os.path.join(HERE, "..", "include", "rtp.h")]

    def compile_one(src):
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
        headers = host_headers if src == "rtp_host.cpp" else kernel_headers
        if force or not _newer(o, [s] + headers):
            cmd = [HIPCC] + FLAGS + ["-c", s, "-o", o]
            tiled = src.startswith(("rtp_gemm_pp_", "rtp_gemm_duo_"))
            if tiled:
                cmd.insert(-4, "-Rpass-analysis=kernel-resource-usage")
                # loops start on an instruction-cache line: left to chance, the same instructions ran up to 10 % slower
                # (256-high tile, 2048 x 1792 x 8192 NN: 137 us starting 28 bytes into a line, 125 us on one)
                cmd.insert(-4, "-falign-loops=64")
                # ... which leaves out loops that are entered in their middle: their first block follows a jump.  (256-high tile of
                # the TN kernel, 4096 x 1376 x 4096: 78.5 us where they fell on a line, 85.0 where the 128 x 128 tile's code had
                # moved them, 80.4 so; 768 x 6144 x 8192 97.3, 103.0, 98.0)
                cmd[-4:-4] = ["-mllvm", "-align-all-nofallthru-blocks=6"]
            if verbose:
                print(" ".join(cmd), flush=True)
            res = subprocess.run(cmd, check=True, stderr=subprocess.PIPE, text=True)
            if tiled:
                # the tiled GEMM must keep its accumulators in registers: a build that spills is a broken build
                spills = [ln for ln in res.stderr.splitlines() if "ScratchSize" in ln and not ln.rstrip().endswith(": 0 [-Rpass-analysis=kernel-resource-usage]")]
                if spills:
                    raise RuntimeError(f"{src}: the tiled GEMM kernel spills registers to scratch memory:\n" + "\n".join(spills))
                # ... and leave room for a wave of the staging copy kernel beside its own two waves on a SIMD (512 registers):
                # above 208 the copies only run where no GEMM wave sits, and the steps wait for them.  (No copies run beside
                # gemm_duo_kernel: its two workgroups may fill the SIMD.)
                import re
                limit = 256 if src.startswith("rtp_gemm_duo_") else 208
                fat = [ln for ln in res.stderr.splitlines() if (m := re.search(r" VGPRs: (\d+)", ln)) and int(m.group(1)) > limit]
                if fat:
                    raise RuntimeError(f"{src}: the tiled GEMM kernel uses more than {limit} vector registers:\n" + "\n".join(fat))
        return o

    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    if force or not _newer(LIB, objs):
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, check=True)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(force="--force" in sys.argv, verbose=True))
