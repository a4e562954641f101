// Which graphs run their rounds as steps of two launches: host code without HIP,
// so that the tests can check the rule by itself.
#pragma once

#include <stdint.h>

namespace pp {

// Late pulls stop lists early on graphs with this many arcs or more: below, a
// round is bound by its launches and the steps' dependent loads add to it
// (undirected R-MAT 13, 512 seeds: 3.9 -> 4.5 ms for its 16 groups; ER 10k: 192 ->
// 204 us; but undirected R-MAT 17, 4M arcs: round 4 96 -> 45 us).  Propagations of
// R-MATs with 16 arcs a node, 64 / 256 / 512 seeds, as steps and with early exits, us:
// 362k arcs 174 / 198 / 222 and 197 / 227 / 282, 923k 194 / 234 / 356 and 208 / 238 / 321,
// 1.5M 211 / 310 / 386 and 222 / 300 / 347, 3.1M 294 / 345 / 483 and 277 / 335 / 387, 6.3M 393 /
// 468 / 716 and 352 / 410 / 532; random graphs cross between 1.5M and 3M as well.
constexpr int64_t EXIT_MIN_ARCS = (int64_t)1 << 20;

// graphs of fewer arcs run their rounds as steps of two launches, as do those
// whose pulls take the short-list form with any number of arcs: three launches
// cost 1-3 us more per round (10,000-node graph of 100,000 arcs, 64 seeds: 184
// -> 174 us; 301^2 lattice 4.80 -> 4.53 ms; 13-scale R-MAT, 512 seeds in two
// groups: 0.99 -> 0.94 ms; 4096^2 lattice, 60M arcs, 128 seeds: 99.3 -> 96.9).
// Larger graphs with long lists have their pushes' occupancy to lose (the
// joint kernel's registers halve it) or early-exit pulls of three launches.
constexpr int64_t STEP_MAX_ARCS = EXIT_MIN_ARCS;

// short_form: the run's pulls take the short-list form; exit_ok: late pulls may
// stop lists early; skip_dead: the general pull leaves the rows of nodes without
// successors alone, a form that the joint kernel does not have, and such graphs
// have rows beyond the caches to gain from it whatever their arcs (20M nodes, 1M
// arcs, 64 and 512 seeds: 1.28 and 4.38 ms in three launches, 1.39 and 6.16 in
// steps; 4M nodes, 512 seeds: 1.95 and 2.27).
inline bool takes_steps(int64_t m, bool short_form, bool exit_ok, bool skip_dead) {
    if (exit_ok) return false;
    return short_form || (m < STEP_MAX_ARCS && !skip_dead);
}

// Whether a single step follows the first batch of steps instead of another batch:
// a step that listed a frontier left the batch a round short, and the new bits
// fell to less than a quarter of the round before's (decay: that ratio, 4 and above
// as 1, a feature of the scheduler), so the propagation is likely to end in it.  A
// small random graph of diameter 7 has eight rounds and one listing (10,000 nodes,
// 256 and 512 seeds: three launches a round 200 and 216 us, 229 and 248 with a batch
// of eight steps behind the first, 196 and 220 with one step; nine steps in every first
// batch instead cost graphs that end sooner 3-6%).
inline bool one_more_step(int64_t listings, float decay) { return listings > 0 && decay < 0.0625f; }

}  // namespace pp
