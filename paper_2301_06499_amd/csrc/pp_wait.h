// When a wait between blocks gives up: host and device code (the tests compile it
// for the host).
#pragma once

#include <stdint.h>

#include "pp_close.h"   // PP_HD

namespace pp {

// A wait of about ten seconds by the 100 MHz clock, and at least a million polls
// (one to two seconds of polling): a wait whose queue was switched out meanwhile
// goes on.  The clock's difference is signed: nothing orders two readings (scalar
// loads may complete out of order, and the first is still in flight when the
// second is issued), and with an unsigned one a single tick backwards is taken for
// a wait of centuries.  The polls alone end a wait whose clock does not advance.
constexpr int64_t WAIT_TICKS = 1000000000;
constexpr uint32_t WAIT_POLLS_MIN = 1u << 20, WAIT_POLLS_MAX = 1u << 26;
struct BoundedWait {
    uint64_t t0;
    uint32_t polls;
    PP_HD bool expired(uint64_t now) {
        ++polls;
        return (polls >= WAIT_POLLS_MIN && (int64_t)(now - t0) > WAIT_TICKS) || polls >= WAIT_POLLS_MAX;
    }
};

}  // namespace pp
