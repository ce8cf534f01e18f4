"""Build the HIP library for gfx950, in-tree: python -m paper_2511_11446_amd.build"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdiffpro_qlinear.so")
SOURCES = ["daq.hip", "daq_robust.hip", "daq_ln.hip", "qgemm.hip", "qgemm_w4.hip", "qgemm_small.hip", "qgemm_big.hip", "qgemm_w4_big.hip", "qgemm_many.hip", "offline_host.hip", "api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    "-ffp-contract=off",                            # every fused multiply-add in the kernels is written out
    "-fhip-fp32-correctly-rounded-divide-sqrt",      # DAQ needs the IEEE quotient
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]

# The K loops of the DMA tiles and of the 4-bit ones begin at a multiple of 16 bytes.  Where they begin otherwise depends on all code in front of them, and a start 4 bytes behind
# a multiple of 8 cost FP16 layers with GELU or gate 1 % (256x192 tiles: M = 2048, K = 1152, N = 4608) to 4 % (64x64: M = 1024, K = 3072, N = 768, 16.9 -> 16.2 us), and 64x64 tiles of
# 4-bit weights up to 5 % (M = 384, K = 4608, N = 1152, 25.0 -> 23.9 us).  Multiples of 64 took 1.3 % from the plain FP16 tiles of 128x128, and the 8-bit kernels of few
# rows (qgemm_small.hip) were 0.3 % slower aligned than not.
FILE_FLAGS = {src: ["-Xarch_device", "-falign-loops=16"] for src in ("qgemm.hip", "qgemm_w4.hip")}


def _compile(src):
    obj = os.path.join(OBJDIR, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        print(out, file=sys.stderr)
    return obj


def build(verbose=True):
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp,
                           "-Wno-unused-command-line-argument"])
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


# bench.py's measurement aid (a register-resident MFMA loop): a shared object of its own beside bench.py, not in the library
PROBE_SRC = os.path.join(os.path.dirname(HERE), "bench_mfma_probe.hip")
PROBE_LIB = os.path.join(os.path.dirname(HERE), "libbench_mfma_probe.so")


def build_bench_probe(verbose=True):
    tmp = PROBE_LIB + ".tmp%d" % os.getpid()
    r = subprocess.run([HIPCC, *FLAGS, "-shared", PROBE_SRC, "-o", tmp], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (PROBE_SRC, r.stdout))
    os.replace(tmp, PROBE_LIB)
    if verbose:
        print("built", PROBE_LIB)
    return PROBE_LIB


if __name__ == "__main__":
    build()
    build_bench_probe()
