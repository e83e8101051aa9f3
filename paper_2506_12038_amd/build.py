"""Build liblcd.so (HIP, gfx950 only) in-tree with hipcc.  No JIT, no torch extension."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
LIB = PKG / "liblcd.so"
BUILD = ROOT / "_build"

SOURCES = ["lcd_host.cpp", "lcd_pack.hip", "lcd_gemv.hip", "lcd_bucket.hip", "lcd_tokens.hip", "lcd_tokens_mixed.hip", "lcd_narrow.hip", "lcd_gemm.hip", "lcd_gemm_split.hip", "lcd_gemm_wide.hip", "lcd_gemm_mixed.hip",
           "lcd_cluster.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    f"-I{ROOT / 'include'}", f"-I{CSRC}",
]


# The prefill kernels (lcd_gemm_*.hip) keep their accumulators in fixed AGPRs through inline assembly: the compiler
# must not use AGPRs as spill space there.
# lcd_pack.hip, lcd_gemv.hip: the same for the transformation of one input.
# lcd_bucket.hip, lcd_tokens.hip, lcd_tokens_mixed.hip: the decode kernels' eleven (twelve) leading arguments (the table of first
# workgroups or a single layer, the input the layers share, the widths' first workgroups) are preloaded into scalar registers at wave start
# instead of being read from the argument segment.
EXTRA = {"lcd_gemm_split.hip": ["-mllvm", "-amdgpu-spill-vgpr-to-agpr=0"],
         "lcd_gemm_wide.hip": ["-mllvm", "-amdgpu-spill-vgpr-to-agpr=0"],
         "lcd_gemm_mixed.hip": ["-mllvm", "-amdgpu-spill-vgpr-to-agpr=0"],
         "lcd_pack.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=10"],
         "lcd_gemv.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=9"],
         "lcd_bucket.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=11"],
         "lcd_tokens.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=11"],
         "lcd_narrow.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=11"],
         "lcd_tokens_mixed.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=12"]}


# Sources that are compiled once for each index width, side by side (one after the other they take minutes).
EACH_WIDTH = ("lcd_gemm_wide.hip", "lcd_gemm_mixed.hip")


def _compile(src: str, width: int, keep_asm: bool) -> Path:
    # a folder for each job: kept temporaries are named after the source alone
    name = src.rsplit(".", 1)[0] + (f"_{width}" if width else "")
    folder = BUILD / name
    folder.mkdir(parents=True, exist_ok=True)
    obj = folder / (name + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), *([f"-DLCD_GEMM_BITS={width}"] if width else []), "-c", str(CSRC / src), "-o", str(obj)]
    if keep_asm and src.endswith(".hip"):
        cmd += ["-save-temps=obj"]
    subprocess.check_call(cmd, cwd=str(folder), stderr=subprocess.DEVNULL if not os.environ.get("LCD_BUILD_VERBOSE") else None)
    return obj


def build_library(keep_asm: bool = False) -> Path:
    """Compile every source and link paper_2506_12038_amd/liblcd.so."""
    srcs = [s for s in SOURCES if (CSRC / s).exists()]
    jobs = sorted(((s, w) for s in srcs for w in ((2, 3, 4) if s in EACH_WIDTH else (0,))), key=lambda j: j[1] == 0)    # (the longest first)
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(lambda j: _compile(*j, keep_asm), jobs))
    tmp = LIB.with_suffix(".so.tmp%d" % os.getpid())
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *map(str, objs), "-o", str(tmp)])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(keep_asm=bool(os.environ.get("LCD_KEEP_ASM"))))
