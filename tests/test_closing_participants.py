"""Which blocks of a round's closing launch take part (pp_close.h, compiled for
the host): a block that the dispatcher starts late, when the block that ends the
round may have rewritten any of the control block's fields, never takes part,
whatever the next round is -- a late block that did would work on the next
round and leave a ticket behind."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "pp_close.h"
// mode values of the kernels: 0 pull, 1 push, 3 sparse pull
struct Block { int32_t converged, round, mode, exit_round, nodes[2], close_round, close_mode; };
// every field a load may find old or new: bit k of `late` chooses for field k
struct Read {
    const Block &a, &b;
    unsigned late;
    const Block &at(int k) const { return (late >> k) & 1 ? b : a; }
    int32_t converged() const { return at(0).converged; }
    int32_t close_round() const { return at(1).close_round; }
    int32_t close_mode() const { return at(2).close_mode; }
    int32_t nodes(int p) const { return at(3 + p).nodes[p]; }
};
int main() {
    const int grid = 64, block = 256, W = 4, modes[3] = {0, 1, 3};
    const int32_t sizes[4] = {0, 3, 700, 100000};
    long cases = 0, wrong = 0;
    for (int mode : modes) for (int next : modes) for (int exit = 0; exit < 2; ++exit) for (int next_exit = 0; next_exit < 2; ++next_exit)
    for (int32_t listed : sizes) for (int32_t hubs : sizes) for (int conv = 0; conv < 2; ++conv) for (int r = 4; r < 6; ++r) {
        const bool ex = mode == 0 && exit;
        Block a{0, r, mode, ex ? r : 0, {0, 0}, 0, 0};
        a.nodes[r & 1] = listed;                  // the round's list
        a.nodes[(r + 1) & 1] = 12345;             // the frontier it pushed
        a.close_round = r;                        // the main launch's note
        a.close_mode = mode | (ex ? pp::CLOSE_EXIT : 0);
        const pp::Closing in = pp::closing(Read{a, a, 0}, hubs, W, grid, block);   // in time
        const long entries = (mode != 0 || ex) ? listed : hubs;
        const long want = (entries * W + block - 1) / block;
        if (in.nb != (want < 1 ? 1 : want > grid ? grid : want) || in.round != r || in.mode != mode) ++wrong;
        Block b = a;                              // after the round's end
        b.converged = conv;
        if (!conv) {
            b.round = r + 1;
            b.mode = next;
            b.exit_round = next_exit ? r + 1 : 0;
            b.nodes[(r + 1) & 1] = 0;
        }
        if (mode == 0) b.nodes[r & 1] = 0;        // what a pull listed
        for (unsigned late = 0; late < 32; ++late) {
            const pp::Closing out = pp::closing(Read{a, b, late}, hubs, W, grid, block);
            ++cases;
            if (out.nb > in.nb) ++wrong;          // a block that should have left would take part
        }
    }
    printf("%ld cases, %ld wrong\n", cases, wrong);
    return wrong != 0;
}
"""


def test_a_late_block_never_takes_part(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "closing.cpp", tmp_path / "closing"
    src.write_text(PROGRAM)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2301_06499_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
