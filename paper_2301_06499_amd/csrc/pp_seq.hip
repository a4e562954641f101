// PROPAGATE-S (Algorithm 2) on gfx950 (wave64): the seeds one at a time with
// one bit per node, k seeds side by side.
//
// Each of the k seeds in flight owns a pair of n-bit signatures (node u is
// bit u & 63 of word u >> 6).  Pass r reads buffer (r-1) & 1 and writes
// buffer r & 1 in full, so the update is synchronous.  A wave takes a word of
// 64 nodes of one seed, one node per lane: a node not reached yet walks its
// successor list and stops at the first successor already reached (the
// algorithm's early break); one ballot gives the word's new bits.  A lane
// walks a short list itself, four arcs per step.  Nodes with more than
// SEQ_LIGHT successors (listed once per graph) are left to a second launch
// in which a group of 32 lanes takes one such node and walks its list 128
// arcs per step up to the first step with a hit, so a hub costs one group,
// not the word that holds it.  Each pass counts, per seed, the nodes it found and
// the arcs it examined (up to and including the first hit of each node); a
// seed is done at its first pass that finds nothing.
//
// That form serves one to seven seeds in flight, and more than 512 on a tiny
// graph (see seq_rows_seeds).  From eight on the same
// passes run on node-major rows of one bit per seed (k_seq_rows), which walk
// each node's list once for all of its seeds; below eight a row of a byte
// would not fit the memory promised (one bit per node, seed and buffer).
#include <mutex>

#include "pp_internal.h"

namespace pp {

#define PS_DEV __device__ __forceinline__

namespace {

PS_DEV int lane() { return __lane_id(); }

PS_DEV bool reached(const uint64_t *sig, int32_t v) { return (sig[v >> 6] >> (v & 63)) & 1ull; }

PS_DEV uint64_t *buffer(const SeqDev &S, int b, int j) {
    return S.bits + ((int64_t)(b & 1) * S.k + j) * S.nw;
}

template <typename T> PS_DEV T block_total(T v, T *scratch) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if (lane() == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    T t = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) t += scratch[w];
    return t;
}

}  // namespace

// Seed j of the batch (kk of them) starts with its own bit; slots kk..k-1
// are idle.  Buffer 0 of every slot was cleared before.
__global__ void __launch_bounds__(BLOCK) k_seq_seeds(SeqDev S, const int32_t *seeds, int kk) {
    for (int j = blockIdx.x * BLOCK + threadIdx.x; j < S.k; j += gridDim.x * BLOCK) {
        S.done[j] = j < kk ? 0 : 1;
        S.dpass[j] = 0;
        S.examined[j] = 0;
        S.pass_cnt[j] = 0;
        if (j < kk) {
            const int32_t x = seeds[j];
            buffer(S, 0, j)[x >> 6] |= 1ull << (x & 63);
        }
        if (j == 0) S.active[0] = kk;
    }
}

// Pass r, nodes with short lists, of every seed still running (grid: blocks
// per seed x k).  Writes every word of the next signature.
__global__ void __launch_bounds__(BLOCK) k_seq_pass(GraphDev g, SeqDev S, int r) {
    const int j = blockIdx.y;
    if (S.done[j]) return;   // the same for the whole block
    const uint64_t *cur = buffer(S, r - 1, j);
    uint64_t *nxt = buffer(S, r, j);
    const int ln = lane();
    const int64_t wave = (int64_t)blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * (BLOCK / 64);
    int64_t found = 0, exam = 0;
    for (int64_t wd = wave; wd < S.nw; wd += nwaves) {   // wave-uniform
        const uint64_t word = cur[wd];
        const int64_t u = wd * 64 + ln;
        const bool open = u < g.n && !((word >> ln) & 1ull);
        int64_t b = 0, e = 0;
        if (open) {
            b = g.rp[u];
            e = g.rp[u + 1];
        }
        bool hit = false;
        if (open && e - b <= SEQ_LIGHT) {   // longer lists: k_seq_heavy
            // the lane's own list, four arcs in flight per step
            for (int64_t a = b; a < e && !hit; a += 4) {
                int32_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = a + q < e ? g.col[a + q] : -1;
                bool t[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) t[q] = v[q] >= 0 && reached(cur, v[q]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (!hit && v[q] >= 0) {
                        ++exam;
                        hit = t[q];
                    }
                }
            }
        }
        const uint64_t nb = __ballot(hit);
        if (ln == 0) {
            nxt[wd] = word | nb;
            found += __popcll(nb);
        }
    }
    __shared__ long long s_red[BLOCK / 64];
    const long long tf = block_total<long long>(found, s_red);
    const long long te = block_total<long long>(exam, s_red);
    if (threadIdx.x == 0) {
        if (tf) atomicAdd((unsigned long long *)&S.pass_cnt[j], (unsigned long long)tf);
        if (te) atomicAdd((unsigned long long *)&S.examined[j], (unsigned long long)te);
    }
}

// Pass r, nodes with long lists (heavy[0..nheavy), stored ids): a group of
// 32 lanes per node, two nodes per wave, each lane four arcs per step (128
// arcs per node and step, in arc order); a hit sets the node's bit in the
// next signature (written by k_seq_pass before, in stream order).  R-MAT 20,
// 256 seeds: 25.3 ms per propagation with 32 lanes, 27.4 with 16, 34.1 with
// 8, 27.5 with 64.
__global__ void __launch_bounds__(BLOCK) k_seq_heavy(GraphDev g, SeqDev S, const int32_t *heavy, int64_t nheavy,
                                                    int r) {
    constexpr int GL = 32;                 // lanes per node
    constexpr int GW = 64 / GL;            // nodes per wave
    const int j = blockIdx.y;
    if (S.done[j]) return;   // the same for the whole block
    const uint64_t *cur = buffer(S, r - 1, j);
    uint64_t *nxt = buffer(S, r, j);
    const int ln = lane();
    const int grp = ln / GL, sub = ln % GL;
    const uint64_t gmask = GL == 64 ? ~0ull : (((1ull << (GL & 63)) - 1) << (grp * GL));
    const int64_t wave = (int64_t)blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * (BLOCK / 64);
    int64_t found = 0, exam = 0;
    for (int64_t h0 = wave * GW; h0 < nheavy; h0 += nwaves * GW) {   // wave-uniform
        const int64_t h = h0 + grp;
        int32_t u = 0;
        bool open = false;
        int64_t b = 0, e = 0;
        if (h < nheavy) {
            u = heavy[h];
            open = !reached(cur, u);
            if (open) {
                b = g.rp[u];
                e = g.rp[u + 1];
            }
        }
        bool hit = false;     // the same in every lane of a group
        int64_t ex = 0;
        for (int64_t a0 = b; __ballot(open && !hit && a0 < e); a0 += 4 * GL) {   // wave-uniform condition
            const bool go = open && !hit && a0 < e;
            bool t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t a = a0 + q * GL + sub;
                t[q] = go && a < e && reached(cur, g.col[a]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t m = (__ballot(t[q]) & gmask) >> (grp * GL);
                if (go && !hit) {
                    if (m) {
                        hit = true;
                        ex += __ffsll((long long)m);   // this chunk's arcs up to the first hit, in arc order
                    } else {
                        const int64_t left = e - (a0 + q * GL);
                        ex += left <= 0 ? 0 : (left < GL ? left : GL);
                    }
                }
            }
        }
        if (sub == 0) {   // one lane per group counts and sets the bit
            exam += ex;
            if (hit) {
                ++found;
                atomicOr((unsigned long long *)&nxt[u >> 6], 1ull << (u & 63));
            }
        }
    }
    __shared__ long long s_red[BLOCK / 64];
    const long long tf = block_total<long long>(found, s_red);
    const long long te = block_total<long long>(exam, s_red);
    if (threadIdx.x == 0) {
        if (tf) atomicAdd((unsigned long long *)&S.pass_cnt[j], (unsigned long long)tf);
        if (te) atomicAdd((unsigned long long *)&S.examined[j], (unsigned long long)te);
    }
}

// After pass r: a seed whose pass found nothing is done; otherwise r is its
// last pass so far with a find.  A seed still running at the last pass the
// log holds is stopped and counted as not converged.
// The pass's finds are summed into sum_cnt[r].
__global__ void __launch_bounds__(BLOCK) k_seq_end(SeqDev S, int r) {
    long long sum = 0;
    for (int j = blockIdx.x * BLOCK + threadIdx.x; j < S.k; j += gridDim.x * BLOCK) {
        if (S.done[j]) continue;
        const int64_t c = S.pass_cnt[j];
        S.pass_cnt[j] = 0;
        sum += c;
        if (c == 0) {
            S.done[j] = 1;
            atomicSub(S.active, 1);
        } else {
            S.dpass[j] = r;
            if (r + 1 >= S.cap) {
                S.done[j] = 2;
                atomicSub(S.active, 1);
            }
        }
    }
    __shared__ long long s_red[BLOCK / 64];
    const long long t = block_total<long long>(sum, s_red);
    if (threadIdx.x == 0 && t) atomicAdd((unsigned long long *)&S.sum_cnt[r], (unsigned long long)t);
}

// ---------------------------------------------------------------- node-major rows

namespace {

template <typename T, int P> PS_DEV void load_slice(const T *p, T (&v)[P]) {
    if constexpr (P == 2) {
        const ulonglong2 q = *reinterpret_cast<const ulonglong2 *>(p);
        v[0] = q.x;
        v[1] = q.y;
    } else {
        v[0] = p[0];
    }
}

template <typename T, int P> PS_DEV void store_slice(T *p, const T (&v)[P]) {
    if constexpr (P == 2) {
        ulonglong2 q;
        q.x = v[0];
        q.y = v[1];
        *reinterpret_cast<ulonglong2 *>(p) = q;
    } else {
        p[0] = v[0];
    }
}

template <typename T, int P> PS_DEV bool any_bit(const T (&v)[P]) {
    T o = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) o |= v[k];
    return o != 0;
}

template <typename T, int P> PS_DEV int bits(const T (&v)[P]) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) c += __popcll((unsigned long long)v[k]);
    return c;
}

template <typename T> PS_DEV T from_lane(T v, int lane_) {
    if constexpr (sizeof(T) == 8) return (T)__shfl((unsigned long long)v, lane_);
    else return (T)__shfl((unsigned int)v, lane_);
}

}  // namespace

// Node u's list, walked by NWV waves (one, or the whole block) in steps of
// NWV x 64 / L x SEQ_STEP consecutive arcs: each group of L lanes (16 bytes of a
// row per lane) gathers SEQ_STEP of them, an exclusive prefix OR over the groups
// (and, through LDS, over the waves) gives every group the bits still pending
// at its first arc, and a step whose rows are all zero skips it.  The new row
// goes to nxt.  Bound by the chain of steps of the longest lists, which is why
// they take a block (R-MAT 20, 256 seeds, passes 1 and 2, which walk every list to
// its end: 377 and 324 us with a wave each, 150 and 151 us).
constexpr int SEQ_STEP = 4;
template <typename T, int W, int NWV>
PS_DEV void walk_list(const GraphDev &g, const T *cur, T *nxt, int32_t u, const T *rn, T *gain, int64_t &found,
                      int64_t &exam) {
    constexpr int L = W >= 2 ? W / 2 : 1, P = W / L, NG = 64 / L, ST = SEQ_STEP;
    __shared__ T s_or[2][NWV][W];
    const int ln = lane(), sub = ln % L, grp = ln / L, wv = NWV > 1 ? threadIdx.x >> 6 : 0;
    const int64_t mine = ((int64_t)wv * NG + grp) * ST;   // the group's first arc of a step
    int64_t a = g.rp[u];
    const int64_t e = g.rp[u + 1];
    T row[P], pend[P];
    load_slice<T, P>(cur + (int64_t)u * W + sub * P, row);
#pragma unroll
    for (int k = 0; k < P; ++k) pend[k] = rn[k] & (T)~row[k];
    int32_t v[ST];
#pragma unroll
    for (int q = 0; q < ST; ++q) v[q] = a + mine + q < e ? g.col[a + mine + q] : -1;
    int par = 0;
    while (a < e && __ballot(any_bit<T, P>(pend))) {   // the same in every wave
        T rows[ST][P];
#pragma unroll
        for (int q = 0; q < ST; ++q) {
            if (v[q] >= 0) {
                load_slice<T, P>(cur + (int64_t)v[q] * W + sub * P, rows[q]);
            } else {
#pragma unroll
                for (int k = 0; k < P; ++k) rows[q][k] = 0;
            }
        }
        const int64_t left = e - (a + mine);   // arcs from the group's first on
        a += NWV * NG * ST;
#pragma unroll
        for (int q = 0; q < ST; ++q) v[q] = a + mine + q < e ? g.col[a + mine + q] : -1;
        T o[P], p[P], all[P];   // the groups' ORs up to this one; bits pending here; the step's OR
#pragma unroll
        for (int k = 0; k < P; ++k) {
            o[k] = 0;
#pragma unroll
            for (int q = 0; q < ST; ++q) o[k] |= rows[q][k];
            p[k] = pend[k];
            all[k] = 0;
        }
        if (__ballot(any_bit<T, P>(o))) {   // wave-uniform
#pragma unroll
            for (int k = 0; k < P; ++k) {
#pragma unroll
                for (int d = L; d < 64; d <<= 1) {   // inclusive prefix OR over the groups
                    const T t = from_lane<T>(o[k], ln - d < 0 ? ln : ln - d);
                    o[k] |= t;
                }
                const T before = from_lane<T>(o[k], ln < L ? ln : ln - L);
                p[k] &= (T)~(ln < L ? (T)0 : before);
                all[k] = from_lane<T>(o[k], 64 - L + sub);
            }
        }
        if constexpr (NWV > 1) {   // the waves before this one, and all of them
            if (grp == 0) store_slice<T, P>(&s_or[par][wv][sub * P], all);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < P; ++k) all[k] = 0;
#pragma unroll
            for (int w = 0; w < NWV; ++w) {
                T x[P];
                load_slice<T, P>(&s_or[par][w][sub * P], x);
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    if (w < wv) p[k] &= (T)~x[k];
                    all[k] |= x[k];
                }
            }
            par ^= 1;
        }
#pragma unroll
        for (int k = 0; k < P; ++k) pend[k] &= (T)~all[k];
#pragma unroll
        for (int q = 0; q < ST; ++q) {
            if (q < left) exam += bits<T, P>(p);
#pragma unroll
            for (int k = 0; k < P; ++k) p[k] &= (T)~rows[q][k];
        }
    }
    if (grp == 0 && wv == 0) {
        T nb[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            nb[k] = rn[k] & (T)~row[k] & (T)~pend[k];
            row[k] |= nb[k];
            gain[k] |= nb[k];
        }
        found += bits<T, P>(nb);
        store_slice<T, P>(nxt + (int64_t)u * W + sub * P, row);
    }
    if constexpr (NWV > 1) __syncthreads();   // the LDS words before the next node's
}

// Pass r of every seed in flight on rows of W words of type T (bit i: seed i).
// A node's pending bits are the running seeds that have not reached it; its
// list is walked in order, each arc adds one examined arc per pending bit and
// clears the bits of its successor's row, and the walk ends when none is left:
// each seed's early break at its own first hit, counted as if it walked alone.
// The first giant_blocks blocks take the nodes with more than SEQ_GIANT
// successors, one per block, the next heavy_blocks those with more than
// SEQ_LIGHT, one per wave (walk_list); the other blocks take the rest, one node
// per group of L lanes.  Every node's row goes to the next buffer.
// Bound by the gathers of a dense round (one row per arc serves every seed),
// like the pull of PROPAGATE-P; the seed-major form gathers a word per arc and
// seed.  R-MAT 20, 256 seeds, per call: 22.8 ms seed-major (two launches of
// passes, 22.1 ms in them), 0.87 ms here (0.82 ms in the passes).
template <typename T, int W>
__global__ void __launch_bounds__(BLOCK) k_seq_rows(GraphDev g, SeqRows S, const int32_t *heavy, int64_t nheavy,
                                                   int64_t ngiant, int r, int giant_blocks, int heavy_blocks) {
    constexpr int L = W >= 2 ? W / 2 : 1;   // lanes per row
    constexpr int P = W / L;                // words per lane
    constexpr int NG = 64 / L;              // groups per wave
    constexpr int ST = SEQ_STEP;
    const T *cur = (const T *)S.rows + (int64_t)((r - 1) & 1) * g.n * W;
    T *nxt = (T *)S.rows + (int64_t)(r & 1) * g.n * W;
    const unsigned long long *run = S.run + ((r - 1) % 3) * SEQ_WORDS;   // the seeds that found a node in pass r - 1
    unsigned long long *found_by = S.run + (r % 3) * SEQ_WORDS;
    if (blockIdx.x == 0 && threadIdx.x < SEQ_WORDS) S.run[((r + 1) % 3) * SEQ_WORDS + threadIdx.x] = 0;
    const int ln = lane(), sub = ln % L, grp = ln / L, wv = threadIdx.x >> 6;
    T rn[P];
    bool open_seeds = false;
#pragma unroll
    for (int w = 0; w < W; ++w) open_seeds |= run[w] != 0;
    if (!open_seeds) return;   // every seed is done
#pragma unroll
    for (int k = 0; k < P; ++k) rn[k] = (T)run[sub * P + k];
    int64_t found = 0, exam = 0;
    T gain[P];
#pragma unroll
    for (int k = 0; k < P; ++k) gain[k] = 0;

    if ((int)blockIdx.x < giant_blocks) {
        for (int64_t h = blockIdx.x; h < ngiant; h += giant_blocks)   // block-uniform
            walk_list<T, W, BLOCK / 64>(g, cur, nxt, heavy[h], rn, gain, found, exam);
    } else if ((int)blockIdx.x < giant_blocks + heavy_blocks) {
        const int64_t nw = (int64_t)heavy_blocks * (BLOCK / 64);
        for (int64_t h = ngiant + (int64_t)(blockIdx.x - giant_blocks) * (BLOCK / 64) + wv; h < nheavy; h += nw)   // wave-uniform
            walk_list<T, W, 1>(g, cur, nxt, heavy[h], rn, gain, found, exam);
    } else {
        const int before = giant_blocks + heavy_blocks;
        const int64_t nw = (int64_t)(gridDim.x - before) * (BLOCK / 64);
        const int64_t first = (int64_t)(blockIdx.x - before) * (BLOCK / 64) + wv;
        for (int64_t u0 = first * NG; u0 < g.n; u0 += nw * NG) {   // wave-uniform
            const int64_t u = u0 + grp;
            int64_t a = 0;
            int64_t left = 0;
            bool mine = u < g.n;
            T row[P], pend[P];
#pragma unroll
            for (int k = 0; k < P; ++k) row[k] = 0;
            if (mine) {
                a = g.rp[u];
                left = g.rp[u + 1] - a;
                load_slice<T, P>(cur + u * W + sub * P, row);
            }
            mine = mine && left <= SEQ_LIGHT;
#pragma unroll
            for (int k = 0; k < P; ++k) pend[k] = mine ? (T)(rn[k] & (T)~row[k]) : (T)0;
            while (true) {   // wave-uniform exit
                const uint64_t m = __ballot(any_bit<T, P>(pend) && left > 0);
                if (m == 0) break;
                const bool go = ((m >> (ln - sub)) & ((1ull << L) - 1ull)) != 0;   // any lane of the group
                int32_t v[ST];
#pragma unroll
                for (int q = 0; q < ST; ++q) v[q] = go && q < left ? g.col[a + q] : -1;
                T rows[ST][P];
#pragma unroll
                for (int q = 0; q < ST; ++q) {
                    if (v[q] >= 0) {
                        load_slice<T, P>(cur + (int64_t)v[q] * W + sub * P, rows[q]);
                    } else {
#pragma unroll
                        for (int k = 0; k < P; ++k) rows[q][k] = 0;
                    }
                }
#pragma unroll
                for (int q = 0; q < ST; ++q) {
                    if (v[q] >= 0) exam += bits<T, P>(pend);
#pragma unroll
                    for (int k = 0; k < P; ++k) pend[k] &= (T)~rows[q][k];
                }
                a += ST;
                left -= ST;
            }
            if (mine) {
                T nb[P];
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    nb[k] = rn[k] & (T)~row[k] & (T)~pend[k];
                    row[k] |= nb[k];
                    gain[k] |= nb[k];
                }
                found += bits<T, P>(nb);
                store_slice<T, P>(nxt + u * W + sub * P, row);
            }
        }
    }
    // the block's sums; a seed that found a node runs on (bits only get set, so
    // a block whose bits are all there adds nothing)
    __shared__ long long s_red[BLOCK / 64];
    __shared__ unsigned long long s_gain[SEQ_WORDS];
    if (threadIdx.x < SEQ_WORDS) s_gain[threadIdx.x] = 0;
    const long long tf = block_total<long long>(found, s_red);   // its barriers order the clears
    const long long te = block_total<long long>(exam, s_red);
#pragma unroll
    for (int k = 0; k < P; ++k) {
        unsigned long long o = (unsigned long long)gain[k];
#pragma unroll
        for (int d = 32; d >= L; d >>= 1) o |= __shfl_xor(o, d);
        if (grp == 0 && o) atomicOr(&s_gain[sub * P + k], o);
    }
    __syncthreads();
    if (threadIdx.x < W) {
        const unsigned long long o = s_gain[threadIdx.x];
        if (o & ~__hip_atomic_load(&found_by[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicOr(&found_by[threadIdx.x], o);
    }
    if (threadIdx.x == 0) {
        if (tf) atomicAdd((unsigned long long *)&S.sum_cnt[r], (unsigned long long)tf);
        if (te) atomicAdd((unsigned long long *)S.examined, (unsigned long long)te);
    }
}

// Seed j of the batch (kk of them) starts with its own bit, in buffer 0
// (cleared before); the running seeds of pass 1 are all of them.
__global__ void __launch_bounds__(BLOCK) k_seq_rows_seeds(SeqRows S, const int32_t *seeds, int kk) {
    const int W32 = S.row_bytes / 4;   // 32-bit words per row (a narrower row: part of one)
    for (int j = threadIdx.x; j < kk; j += BLOCK) {
        const int64_t byte = (int64_t)seeds[j] * S.row_bytes + (W32 ? (j >> 5) * 4 : 0);
        const int bit = W32 ? j & 31 : j + 8 * (int)(byte & 3);   // a narrow row lies inside its 4-byte word
        atomicOr((unsigned int *)S.rows + (byte >> 2), 1u << bit);
    }
    for (int w = threadIdx.x; w < 3 * SEQ_WORDS; w += BLOCK) {
        const int lo = w * 64;   // seeds of word w of the first mask
        const int c = w < SEQ_WORDS ? (kk - lo < 0 ? 0 : (kk - lo > 64 ? 64 : kk - lo)) : 0;
        S.run[w] = c == 64 ? ~0ull : (1ull << c) - 1ull;
    }
    if (threadIdx.x == 0) *S.examined = 0;
}

hipError_t launch_seq_rows_seeds(const SeqRows &S, const int32_t *seeds, int kk, hipStream_t st) {
    hipLaunchKernelGGL(k_seq_rows_seeds, dim3(1), dim3(BLOCK), 0, st, S, seeds, kk);
    return hipGetLastError();
}

template <typename T, int W>
static hipError_t seq_rows_impl(const GraphDev &g, const SeqRows &S, const int32_t *heavy, int64_t nheavy,
                                int64_t ngiant, int r, hipStream_t st) {
    constexpr int NG = 64 / (W >= 2 ? W / 2 : 1);
    const int64_t hb = (nheavy - ngiant + BLOCK / 64 - 1) / (BLOCK / 64), lb = (g.n + NG * (BLOCK / 64) - 1) / (NG * (BLOCK / 64));
    const int nh = (int)(hb < SEQ_BLOCKS ? hb : SEQ_BLOCKS), nl = (int)(lb < SEQ_BLOCKS ? lb : SEQ_BLOCKS);
    const int ng = (int)(ngiant < SEQ_BLOCKS ? ngiant : SEQ_BLOCKS);
    hipLaunchKernelGGL((k_seq_rows<T, W>), dim3(ng + nh + nl), dim3(BLOCK), 0, st, g, S, heavy, nheavy, ngiant, r, ng, nh);
    return hipGetLastError();
}

hipError_t launch_seq_rows(const GraphDev &g, const SeqRows &S, const int32_t *heavy, int64_t nheavy, int64_t ngiant,
                           int r, hipStream_t st) {
    switch (S.row_bytes) {
        case 1: return seq_rows_impl<uint8_t, 1>(g, S, heavy, nheavy, ngiant, r, st);
        case 2: return seq_rows_impl<uint16_t, 1>(g, S, heavy, nheavy, ngiant, r, st);
        case 4: return seq_rows_impl<uint32_t, 1>(g, S, heavy, nheavy, ngiant, r, st);
        case 8: return seq_rows_impl<uint64_t, 1>(g, S, heavy, nheavy, ngiant, r, st);
        case 16: return seq_rows_impl<uint64_t, 2>(g, S, heavy, nheavy, ngiant, r, st);
        case 32: return seq_rows_impl<uint64_t, 4>(g, S, heavy, nheavy, ngiant, r, st);
        case 64: return seq_rows_impl<uint64_t, 8>(g, S, heavy, nheavy, ngiant, r, st);
        default: return hipErrorInvalidValue;
    }
}

// The fixed device region of pp_propagate_s_noalloc: PROPAGATE-S's buffers
// for callers that cannot allocate.  Every device the library runs on holds
// its own copy, at its own address, until the process ends.  Host code never
// passes the array's name to a kernel (on the host it only stands for the
// symbol): it takes the device address from hipGetSymbolAddress once per
// device and passes that.
static __device__ __align__(256) unsigned char scratch[PP_NOALLOC_BYTES];

namespace {
constexpr int MAX_DEVICES = 256;
std::mutex &region_mu() {
    static std::mutex *m = new std::mutex();   // lives until the process ends
    return *m;
}
void *g_region[MAX_DEVICES];   // device address of `scratch` per device (NULL: not looked up yet)
}  // namespace

int noalloc_region(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return set_error(PP_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEVICES) return set_error(PP_EDEVICE, "device %d beyond the %d the library tracks", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lk(region_mu());
    if (!g_region[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return set_error(PP_EDEVICE, "address of the fixed region on device %d: %s", dev, hipGetErrorString(e));
        g_region[dev] = ptr;
    }
    *out = g_region[dev];
    return PP_OK;
}

static int small_grid(int64_t items) {
    const int64_t b = (items + BLOCK - 1) / BLOCK;
    return (int)(b < 1 ? 1 : (b > 1024 ? 1024 : b));
}

hipError_t launch_seq_seeds(const SeqDev &S, const int32_t *seeds, int kk, hipStream_t st) {
    hipLaunchKernelGGL(k_seq_seeds, dim3(small_grid(S.k)), dim3(BLOCK), 0, st, S, seeds, kk);
    return hipGetLastError();
}

hipError_t launch_seq_pass(const GraphDev &g, const SeqDev &S, const int32_t *heavy, int64_t nheavy, int r,
                           int blocks_per_seed, int heavy_blocks_per_seed, hipStream_t st) {
    hipLaunchKernelGGL(k_seq_pass, dim3(blocks_per_seed, S.k), dim3(BLOCK), 0, st, g, S, r);
    if (nheavy > 0)
        hipLaunchKernelGGL(k_seq_heavy, dim3(heavy_blocks_per_seed, S.k), dim3(BLOCK), 0, st, g, S, heavy, nheavy, r);
    hipLaunchKernelGGL(k_seq_end, dim3(small_grid(S.k)), dim3(BLOCK), 0, st, S, r);
    return hipGetLastError();
}

}  // namespace pp
