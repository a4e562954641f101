"""The light rounds' index arithmetic (pp_light.h, compiled for the host) where
32 bits run out: a wave of frontier entries whose predecessor lists hold 2^31
arcs and more together, and a small graph behind 2^32 arcs of a batch."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, program):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "light.cpp", tmp_path / "light"
    src.write_text(program)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2301_06499_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_map_positions_of_a_wave(tmp_path):
    """Waves of 64 entries one after the other, the scan as the kernel keeps it
    (32 bits), against sums in 64 bits: no entry lands inside the map that does
    not belong there."""
    run(tmp_path, r"""
#include <stdio.h>
#include "pp_light.h"
int main() {
    const int H = 4096;
    const uint32_t degs[] = {0, 1, 16, 17, 5000, 1u << 20, 33554432u, 67108863u};
    int wrong = 0;
    for (uint32_t d0 : degs) for (uint32_t d1 : degs) {
        uint64_t base = 0;
        for (int wave = 0; wave < 3; ++wave) {
            uint32_t incl = 0;
            uint64_t at = base;
            for (int ln = 0; ln < 64; ++ln) {
                const uint32_t deg = (ln & 1) ? d1 : d0;
                incl += deg;
                const int want = at < (uint64_t)H ? (int)at : H, got = pp::light_start(base, incl, deg, H);
                wrong += got != want;
                at += deg;
            }
            if (at - base >= 1ull << 32) break;   // a graph of 2^32 arcs takes no light rounds
            base += incl;
            wrong += base != at;
        }
    }
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
""")


def test_arcs_of_a_graph_far_into_a_batch(tmp_path):
    run(tmp_path, r"""
#include <initializer_list>
#include <stdio.h>
#include "pp_light.h"
int main() {
    int wrong = 0;
    for (int64_t first : {(int64_t)0, (int64_t)1 << 31, ((int64_t)1 << 32) - 3, (int64_t)1 << 32, (int64_t)5000000000})
        for (int64_t at : {(int64_t)0, (int64_t)7, ((int64_t)1 << 32) - 20})
            for (int arc : {100, 103, 115})
                wrong += pp::light_arc(first, pp::light_offset(first + at, first), arc, 100) != first + at + (arc - 100);
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
""")
