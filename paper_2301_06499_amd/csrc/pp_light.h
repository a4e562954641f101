// Index arithmetic of the light rounds (light_rounds): host and device code, so
// that the tests can check it on graphs far larger than they can hold.
#pragma once

#include <stdint.h>

#include "pp_close.h"   // PP_HD

namespace pp {

// First flat arc of a frontier entry with deg arcs, at most H (none of its arcs
// then fits the map of arcs): base, the arcs that earlier waves placed; incl, the
// wave's inclusive sum of degrees.  The lists of distinct nodes are disjoint, so
// on a graph of fewer than 2^32 arcs the wave's sum fits 32 bits unsigned (not
// signed).
PP_HD int light_start(uint64_t base, uint32_t incl, uint32_t deg, int H) {
    const uint64_t at = base + (incl - deg);
    return at < (uint64_t)H ? (int)at : H;
}

// First predecessor arc of a node as the frontier in LDS keeps it: from the
// view's first arc, since a batch may hold 2^32 arcs and more where each of its
// graphs holds fewer.
PP_HD uint32_t light_offset(int64_t beg, int64_t view_first) { return (uint32_t)(beg - view_first); }
PP_HD int64_t light_arc(int64_t view_first, uint32_t offset, int32_t arc, int32_t start) {
    return view_first + offset + (arc - start);
}

}  // namespace pp
