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

}  // namespace pp
