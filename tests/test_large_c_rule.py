"""Which problems have their C read and written with the non-temporal hint (csrc/gemm_device.h: c_once):
the rule itself, compiled for the host.  C = A B + C into one C again and again has to find C in the
last-level cache where it fits, so the hint is for a C that does not."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (c_is_f16, M, N, K, ldc, address of C, hint?)
RULE = [
    # measured slower with the hint when one C is used again (16 to 43 %)
    (0, 6000, 6000, 1000, 6000, 1 << 20, 0), (0, 6142, 4720, 216, 4720, 1 << 20, 0), (0, 16169, 3008, 272, 3008, 1 << 20, 0),
    (0, 4774, 12480, 512, 12480, 1 << 20, 0), (1, 4084, 14656, 64, 14656, 1 << 20, 0), (0, 16384, 2304, 768, 2304, 1 << 20, 0),
    # beyond the cache, but with hardly any k loop: still slower (6 to 12 %)
    (0, 4080, 18944, 64, 18944, 1 << 20, 0), (1, 12020, 14144, 128, 14144, 1 << 20, 0),
    # the line: 300 MB, 256 <= K < 4096
    (0, 9155, 8192, 256, 8192, 1 << 20, 0), (0, 9156, 8192, 256, 8192, 1 << 20, 1), (1, 18311, 8192, 1024, 8192, 1 << 20, 1),
    (1, 18310, 8192, 1024, 8192, 1 << 20, 0), (0, 10240, 8192, 248, 8192, 1 << 20, 0), (0, 10240, 8192, 4088, 8192, 1 << 20, 1),
    (0, 10240, 8192, 4096, 8192, 1 << 20, 0),
    # rows of C have to begin at 64-byte sectors
    (0, 10240, 8192, 1024, 8200, 1 << 20, 0), (0, 10240, 8192, 1024, 8208, 1 << 20, 1), (0, 10240, 8192, 1024, 8192, (1 << 20) + 16, 0),
    (1, 20480, 8192, 1024, 8208, 1 << 20, 0), (1, 20480, 8192, 1024, 8224, 1 << 20, 1),
]


def test_hint_on_c(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    src = tmp_path / "rule.hip"
    src.write_text('''
#include "gemm_device.h"
#include <cstdio>
int main() {
    const long long t[][6] = {%s};
    for (auto& r : t) {
        GemmArgs a = {};
        a.c_is_f16 = (int)r[0]; a.M = r[1]; a.N = r[2]; a.K = r[3]; a.ldc = r[4]; a.C = (void*)(uintptr_t)r[5];
        printf("%%d\\n", (int)gemm_dev::c_once(a));
    }
}
''' % ", ".join("{%s}" % ", ".join(str(x) + "LL" for x in row[:6]) for row in RULE))
    exe = tmp_path / "rule"
    subprocess.run(["hipcc", "-std=c++17", "--offload-host-only", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "paper_2108_13191_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]
    assert got == [row[6] for row in RULE], [(row, g) for row, g in zip(RULE, got) if row[6] != g]
