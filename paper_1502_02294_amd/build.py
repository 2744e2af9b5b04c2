"""Build the HIP library liblc.so for gfx950 in-tree (hipcc, no JIT cache).

Every HIP translation unit is compiled with the packed-FP32 target feature
switched off (the compiler still emits scalar FP32 code).
"""
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblc.so")

# (source, object, defines): the fused z pass is compiled per group of grid
# sides, the longest units first
UNITS = [("lc_fused.hip", f"lc_fused{i}.o", [f"-DLC_FUSED_SET={i}"]) for i in (3, 2, 5, 4, 0, 1)] + \
        [("lc_xy.hip", "lc_xy.o", []), ("lc_fft.hip", "lc_fft.o", []), ("lc_dct.hip", "lc_dct.o", []),
         ("lc_field.hip", "lc_field.o", []), ("lc_greens.hip", "lc_greens.o", []), ("lc_host.cpp", "lc_host.o", [])]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-fno-fast-math",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          "-Wno-unused-command-line-argument"]


def _compile(unit, verbose: bool) -> str:
    src, obj, defines = unit
    obj = os.path.join(BUILD, obj)
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = [HIPCC] + COMMON + defines + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda u: _compile(u, verbose), UNITS))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
