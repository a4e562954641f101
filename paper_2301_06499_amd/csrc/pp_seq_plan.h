// How many seeds PROPAGATE-S runs at a time and the device memory that takes:
// host code without HIP, so that the tests can check the rule by itself.
#pragma once

#include <stdint.h>

namespace pp {

constexpr int SEQ_WORDS = 8;   // 64-bit words of the widest node-major row

inline int64_t seq_up(int64_t bytes) { return (bytes + 255) & ~(int64_t)255; }

// One device region holds every buffer of a PROPAGATE-S call for k seeds in
// flight over nw = ceil(n/64) words and a pass log of cap entries (each part
// 256-byte aligned): both signatures of every seed, per-seed pass counts,
// the pass log, per-seed arcs examined, states, last passes, the count of
// running seeds, and the device copy of the batch's seed ids.
inline int64_t seq_region_bytes(int64_t k, int64_t nw, int64_t cap) {
    return seq_up(16 * k * nw) + seq_up(8 * k) + seq_up(8 * cap) + seq_up(8 * k) + seq_up(4 * k) + seq_up(4 * k) +
           seq_up(4) + seq_up(4 * k);
}

// The same for node-major rows of kb seeds: both buffers of rows, the running
// seeds of three passes, the pass log, the arcs examined and the seed ids.
inline int64_t seq_rows_bytes(int64_t n, int kb, int64_t cap) {
    return seq_up(2 * n * (kb / 8)) + seq_up(8 * 3 * SEQ_WORDS) + seq_up(8 * cap) + seq_up(8) + seq_up(4 * kb);
}

// Rows of at most this many bytes in all may hold more seeds than were asked for.
constexpr int64_t SEQ_SMALL_BYTES = (int64_t)4 << 20;

// Seeds at a time on node-major rows when k were asked for, 0 for the seed-major
// form (fewer than eight, or far more than a row holds on a tiny graph).  Rows hold 8, 16, 32, ... 512 seeds.  The most that is
// at most k fits the memory of k one-bit-per-node signature pairs; the least that
// is at least k takes up to twice that, and is used where the caller left the
// number open (roomy) or the rows are small.  A second batch for the seeds that
// are left over costs a small graph as much as the first: 10,000 nodes, 9 to 15
// seeds, 255 us in two batches, 136 us in one, 214 us seed-major; 31 seeds 263, 141
// and 255 us.
// Above 512 a call takes a batch per 512 seeds, each bound by its launches on a
// tiny graph, while the seed-major form takes one, of about a quarter more and
// 7.6e-8 of a batch per seed and item (node or arc): 9000 items, 700 and 4000 seeds,
// 230 and 543 us seed-major, 281 and 1096 in rows; 27,000 items, 359 and 1236
// against 297 and 1167; 2000-node path, 4000 seeds, 89 and 155 ms.
inline int seq_rows_seeds(int64_t k, int64_t n, int64_t m, int64_t cap, bool roomy) {
    if (k < 8) return 0;
    if ((double)((k + 64 * SEQ_WORDS - 1) / (64 * SEQ_WORDS)) > 1.25 + 7.6e-8 * (double)(n + m) * (double)k) return 0;
    int kb = 8;
    while (kb < 64 * SEQ_WORDS && 2 * (int64_t)kb <= k) kb *= 2;
    if (kb < k && kb < 64 * SEQ_WORDS && (roomy || seq_rows_bytes(n, 2 * kb, cap) <= SEQ_SMALL_BYTES)) kb *= 2;
    return kb;
}

}  // namespace pp
