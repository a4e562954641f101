"""How many seeds PROPAGATE-S takes at a time (pp_seq_plan.h, compiled for the
host): one batch for any number of seeds up to 256 where the caller left the
number open or the rows are small, and never more memory than promised."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "pp_seq_plan.h"
int main() {
    int wrong = 0;
    for (int64_t n : {(int64_t)1, (int64_t)63, (int64_t)1000, (int64_t)90601, (int64_t)1 << 20, (int64_t)300000007})
    for (int64_t cap : {(int64_t)1, (int64_t)256, (int64_t)1 << 20})
    for (int64_t k = 1; k <= 1100; ++k)
    for (int roomy = 0; roomy < 2; ++roomy) {
        const int kb = pp::seq_rows_seeds(k, n, 8 * n, cap, roomy);
        if (k < 8) { wrong += kb != 0; continue; }
        if (kb == 0) { wrong += k <= 512 || n > 3000; continue; }   // a tiny graph, more seeds than a row holds
        if (k > 512 && n <= 1000 && k <= 900) { ++wrong; continue; }
        wrong += kb < 8 || kb > 512 || (kb & (kb - 1)) != 0;
        const int64_t promised = pp::seq_region_bytes(k, (n + 63) / 64, cap), rows = pp::seq_rows_bytes(n, kb, cap);
        if (kb > k) wrong += kb >= 2 * k || !(roomy ? rows <= 2 * promised : rows <= 4 << 20);
        else wrong += rows > promised || kb * 2 <= (k < 512 ? k : 512);
        if (roomy && k <= 256) wrong += kb < k;                   // one batch
        if (n <= 1000 && k <= 512 && cap <= 256) wrong += kb < k;   // a small graph's too
    }
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
"""


def test_seeds_at_a_time(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text("#include <initializer_list>\n" + PROGRAM)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2301_06499_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
