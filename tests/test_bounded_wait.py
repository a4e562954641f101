"""When a wait between blocks gives up (pp_wait.h, compiled for the host): not on
a clock that steps back or jumps, not after a pause, but always in the end."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "pp_wait.h"
// polls until the wait gives up when poll k reads clock(k), at most `most`
template <typename F> static uint32_t until(uint64_t t0, uint32_t most, F clock) {
    pp::BoundedWait w{t0, 0};
    for (uint32_t k = 1; k <= most; ++k)
        if (w.expired(clock(k))) return k;
    return 0;
}
int main() {
    int wrong = 0;
    const uint64_t t0 = 77000000000ull;
    const uint32_t day = 1u << 18;   // polls of an ordinary wait, and more
    wrong += until(t0, day, [&](uint32_t k) { return t0 + 100 * (uint64_t)k; }) != 0;
    wrong += until(t0, day, [&](uint32_t) { return t0 - 1; }) != 0;                                // one tick back
    wrong += until(t0, day, [&](uint32_t k) { return k == 5 ? t0 - 12345 : t0 + k; }) != 0;        // once
    wrong += until(t0, day, [&](uint32_t k) { return k == 5 ? t0 + (1ull << 32) : t0 + k; }) != 0; // a carry read early
    wrong += until(t0, day, [&](uint32_t k) { return t0 + 5000000000ull + k; }) != 0;              // switched out for 50 s
    // a wait that never ends is given up after ten seconds: about seven million polls of 1.5 us
    const uint32_t gone = until(t0, 1u << 27, [&](uint32_t k) { return t0 + 150 * (uint64_t)k; });
    wrong += gone < 6000000 || gone > 7000000;
    // and whatever the clock does
    wrong += until(t0, 1u << 27, [&](uint32_t) { return t0; }) == 0;
    wrong += until(t0, 1u << 27, [&](uint32_t) { return t0 - 9; }) == 0;
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
"""


def test_the_wait_gives_up_only_in_the_end(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(PROGRAM)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2301_06499_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
