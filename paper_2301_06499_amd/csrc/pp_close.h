// Which blocks of a round's closing launch (k_post) take part, and what they
// work on.  Host and device code: the tests compile it for the host.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define PP_HD __host__ __device__ __forceinline__
#else
#define PP_HD inline
#endif

namespace pp {

// The closing launch's note of its round: the round's direction, and this bit
// when it is a pull that stops lists early.
constexpr int32_t CLOSE_EXIT = 8;

// Blocks of a closing launch of nb blocks that items (words to commit or
// combine) keep busy: POST_ITEMS per thread, at least one block.  Blocks
// without items would only add ticket latency, and more than one item per
// thread adds serial passes of dependent loads; one item measured best.
constexpr int POST_ITEMS = 1;
PP_HD int post_blocks(int64_t items, int nb, int block) {
    const int64_t b = (items + (int64_t)block * POST_ITEMS - 1) / ((int64_t)block * POST_ITEMS);
    return b < 1 ? 1 : (b < nb ? (int)b : nb);
}

// The round a closing launch of `grid` blocks ends: blocks [0, nb) take part.
struct Closing {
    int32_t round, mode;
    bool list;        // works on the round's list (else on the high-degree nodes)
    int32_t entries;  // of either
    int nb;           // 0: no round ran
};

// The blocks past nb take no ticket, so the block that ends the round may have
// rewritten the control block before a block that the dispatcher starts late
// reads it: of the fields that the round's end writes, a late block must read
// none that could make it take part.  So the round and its direction are the
// note that the round's main launch left (close_round, close_mode), which no
// closing launch writes; converged only ever goes to 1, upon which a block
// leaves; and the list of the round's own parity only ever goes to 0 (after a
// pull), which leaves block 0 alone.
// read: the control block's fields (converged(), close_round(), close_mode(),
// nodes(p)).
template <typename Read> PP_HD Closing closing(const Read &read, int32_t nhubs, int W, int grid, int block) {
    Closing c{0, 0, false, 0, 0};
    if (read.converged()) return c;
    const int32_t note = read.close_mode();
    c.round = read.close_round();
    c.mode = note & (CLOSE_EXIT - 1);
    c.list = c.mode != 0 /* MODE_PULL */ || (note & CLOSE_EXIT);
    c.entries = c.list ? read.nodes(c.round & 1) : nhubs;
    c.nb = post_blocks((int64_t)c.entries * W, grid, block);
    return c;
}

}  // namespace pp
