"""Which graphs run their rounds as steps of two launches (pp_steps.h, compiled
for the host)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "pp_steps.h"
int main() {
    int wrong = 0;
    for (int64_t m : {(int64_t)0, (int64_t)100000, pp::STEP_MAX_ARCS - 1, pp::STEP_MAX_ARCS, (int64_t)60000000})
        for (int f = 0; f < 8; ++f) {
            const bool short_form = f & 1, exit_ok = f & 2, skip_dead = f & 4, steps = pp::takes_steps(m, short_form, exit_ok, skip_dead);
            if (exit_ok) wrong += steps;                                  // early-exit pulls take three launches
            else if (short_form) wrong += !steps;                         // any size
            else wrong += steps != (m < pp::STEP_MAX_ARCS && !skip_dead); // the joint kernel copies dead rows
        }
    // one step behind the first batch: only where a listing left it short of a
    // round, and the new bits are running out
    wrong += pp::one_more_step(0, 0.0f) || pp::one_more_step(1, 0.25f) || pp::one_more_step(1, 1.0f);
    wrong += !pp::one_more_step(1, 0.01f) || !pp::one_more_step(3, 0.0f);
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
"""


def test_steps_rule(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "steps.cpp", tmp_path / "steps"
    src.write_text("#include <initializer_list>\n" + PROGRAM)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2301_06499_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
