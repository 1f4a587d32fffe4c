"""Build the HIP libraries in-tree for gfx950 with hipcc.

libgemm_f16.so         the product: the C ABI of include/gemm_f16.h and the kernels it selects
_fastcall.*.so         the binding's way into the product's entry points without ctypes (csrc/fastcall.c, host code only)
libgemm_f16_ladder.so  the same sources compiled with -DGEMM_F16_LADDER plus csrc/ladder/*.hip: the
                       comparison kernels and ablation rows appended to the configuration table
                       (never selected; tests and profiles reach them by forcing their ids)
"""
from __future__ import annotations

import concurrent.futures
import contextlib
import os
import re
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgemm_f16.so")
FASTCALL = os.path.join(HERE, "_fastcall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
FASTCALL_CC = ("gcc", "cc", "amdclang", "clang")         # the first one that is there (hipcc would link the HIP runtime into it)
LADDER_LIB = os.path.join(HERE, "libgemm_f16_ladder.so")
SOURCES = ["gemm_api.hip", "gemm_generic.hip", "gemm_unaligned.hip", "gemm_unaligned_pp.hip", "gemm_kslice.hip", "gemm_tiled.hip", "gemm_pingpong.hip", "gemm_pp128.hip", "gemm_w4a.hip", "gemm_w4a128.hip", "gemm_splitk_f16.hip"]
LADDER_SOURCES = ["ladder/gemm_w4.hip", "ladder/gemm_overlap.hip", "ladder/gemm_interleaved.hip"]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         # packed-f32 VALU forms are kept off for every HIP file of this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _compile(src: str, obj: str, extra, verbose: bool) -> str:
    cmd = ["hipcc", *FLAGS, *extra, "-c", "-o", obj, os.path.join(CSRC, src)]
    if verbose:
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return res.stdout + res.stderr


def build_fastcall() -> bool:
    """The binding works without it (through ctypes, a microsecond a call slower): what keeps it from being built is
    printed and is no error, and no older build of it stays behind, whose C signatures could be others."""
    with contextlib.suppress(FileNotFoundError):
        os.remove(FASTCALL)
    include = sysconfig.get_paths()["include"]
    cc = next(filter(None, map(shutil.which, FASTCALL_CC)), None)
    if not os.path.exists(os.path.join(include, "Python.h")):
        why = f"no Python.h in {include}"
    elif cc is None:
        why = "no C compiler"
    else:
        res = subprocess.run([cc, "-O2", "-Wall", "-std=c11", "-fPIC", "-shared", "-I" + include, "-o", FASTCALL, os.path.join(CSRC, "fastcall.c")],
                             capture_output=True, text=True)
        sys.stderr.write(res.stderr)
        if res.returncode == 0:
            return True
        why = f"{cc} failed"
    print(f"the binding will call through ctypes: {why}")
    return False


def build(verbose: bool = False, ladder: bool = True, extra=()) -> str:
    """Compile every source (in parallel) and link the product library and, with `ladder`,
    the ladder library.  Returns the product library's path."""
    os.makedirs(OBJ, exist_ok=True)
    jobs = [(s, os.path.join(OBJ, s.replace("/", "_") + ".o"), list(extra)) for s in SOURCES]
    if ladder:
        jobs += [(s, os.path.join(OBJ, s.replace("/", "_") + ".ladder.o"), ["-DGEMM_F16_LADDER", *extra])
                 for s in SOURCES + LADDER_SOURCES]
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        logs = list(pool.map(lambda j: _compile(j[0], j[1], j[2], verbose), jobs))
    link = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-Wno-unused-command-line-argument"]
    subprocess.run([*link, "-o", LIB, *[j[1] for j in jobs[:len(SOURCES)]]], check=True)
    if ladder:
        subprocess.run([*link, "-o", LADDER_LIB, *[j[1] for j in jobs[len(SOURCES):]]], check=True)
    build_fastcall()
    if verbose:
        print(resource_table("".join(logs[:len(SOURCES)])))
    return LIB


def resource_table(text: str) -> str:
    rows, cur = [], {}
    for line in text.splitlines():
        m = re.search(r"remark:\s+(.+?) \[-Rpass", line)
        if not m:
            continue
        body = m.group(1).strip()
        if body.startswith("Function Name:"):
            if cur:
                rows.append(cur)
            cur = {"name": body.split(":", 1)[1].strip()}
        elif ":" in body:
            k, v = body.split(":", 1)
            cur[k.strip()] = v.strip()
    if cur:
        rows.append(cur)
    keys = ["VGPRs", "AGPRs", "TotalSGPRs", "ScratchSize [bytes/lane]", "Occupancy [waves/SIMD]",
            "SGPRs Spill", "VGPRs Spill", "LDS Size [bytes/block]"]
    lines = ["kernel | " + " | ".join(k.split(" [")[0] for k in keys)]
    for r in rows:
        name = subprocess.run(["c++filt", r["name"]], capture_output=True, text=True).stdout.strip() or r["name"]
        name = re.sub(r"\(anonymous namespace\)::", "", name)[:70]
        lines.append(name + " | " + " | ".join(r.get(k, "?") for k in keys))
    return "\n".join(lines)


if __name__ == "__main__":
    build(verbose=True)
    print("built", LIB, "and", LADDER_LIB)
