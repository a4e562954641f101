// Adjacency build on the device (Section 3's graph, as Algorithm 1 reads it):
// the successor rows of the arcs -- self-loops and duplicate arcs removed,
// each row sorted -- and their transpose, from arcs already in device memory.
//
// Each arc u -> v becomes one 64-bit key (u << shift | v), with shift the bit
// width of n, so that a radix sort of the keys' low 2 shift bits orders them
// by row, then by column; equal neighbours are then duplicates, and the row
// boundaries give the row offsets.  A self-loop becomes the key of all ones
// in those bits, above every arc's key (the largest id is below 2^shift - 1),
// which sorts last and is dropped.  The storage order (hub-first, chosen on
// the host from the degrees this file counts) is applied by relabelling the
// sorted keys and sorting again; the transpose is the same keys with the
// halves swapped.
// The result is identical, array for array, to the host build.
#include "pp_internal.h"
#include "pp_build.h"

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>

namespace pp {

namespace {

__global__ void __launch_bounds__(BLOCK) k_check_arcs(const int32_t *a, const int32_t *b, int64_t m, int64_t n,
                                                      const int32_t *node_graph, unsigned long long *first_bad) {
    for (int64_t k = blockIdx.x * (int64_t)BLOCK + threadIdx.x; k < m; k += (int64_t)gridDim.x * BLOCK) {
        const int32_t x = a[k], y = b[k];
        bool bad = x < 0 || x >= n || y < 0 || y >= n;
        if (!bad && node_graph) bad = node_graph[x] != node_graph[y];
        if (bad) atomicMin(first_bad, (unsigned long long)k);
    }
}

// Arc k -> key slot k (and m + k for the reverse arc of an undirected edge).
__global__ void __launch_bounds__(BLOCK) k_arc_keys(const int32_t *a, const int32_t *b, int64_t m, int shift,
                                                    bool undirected, uint64_t no_arc, uint64_t *keys) {
    for (int64_t k = blockIdx.x * (int64_t)BLOCK + threadIdx.x; k < m; k += (int64_t)gridDim.x * BLOCK) {
        const uint64_t x = (uint32_t)a[k], y = (uint32_t)b[k];
        const bool loop = x == y;
        keys[k] = loop ? no_arc : (x << shift | y);
        if (undirected) keys[m + k] = loop ? no_arc : (y << shift | x);
    }
}

// Row lengths from the run boundaries of sorted keys: the run of row r adds
// its end index and subtracts its start index, one atomic each per row.
__global__ void __launch_bounds__(BLOCK) k_row_lengths(const uint64_t *keys, int64_t count, int shift,
                                                       unsigned long long *len) {
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
        const uint64_t r = keys[i] >> shift;
        if (i == 0 || (keys[i - 1] >> shift) != r) atomicAdd(&len[r], (unsigned long long)(0 - (uint64_t)i));
        if (i == count - 1 || (keys[i + 1] >> shift) != r) atomicAdd(&len[r], (unsigned long long)(i + 1));
    }
}

__global__ void __launch_bounds__(BLOCK) k_key_cols(const uint64_t *keys, int64_t count, uint64_t mask, int32_t *col) {
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK)
        col[i] = (int32_t)(keys[i] & mask);
}

// Run lengths of sorted columns (in-degrees): each run's end adds its index + 1,
// its start takes its index away.
__global__ void __launch_bounds__(BLOCK) k_col_counts(const uint32_t *cols, int64_t count, int32_t *cnt) {
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
        const uint32_t c = cols[i];
        const bool first = i == 0 || cols[i - 1] != c, last = i == count - 1 || cols[i + 1] != c;
        if (first || last)   // (sums of 32 bits: a column's count fits, its indices may wrap)
            atomicAdd(&cnt[c], (last ? (int32_t)(uint32_t)(i + 1) : 0) - (first ? (int32_t)(uint32_t)i : 0));
    }
}

// The same of columns in any order, where there is no memory to sort them.
__global__ void __launch_bounds__(BLOCK) k_col_adds(const uint32_t *cols, int64_t count, int32_t *cnt) {
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK)
        atomicAdd(&cnt[cols[i]], 1);
}

// ---- the storage order on the device (device_order below)

// Nodes with in-degree at least thr: sort key (in-degree descending, id).
__global__ void __launch_bounds__(BLOCK) k_hot_keys(const int32_t *indeg, int64_t n, double thr, uint64_t *keys,
                                                    unsigned int *count) {
    for (int64_t v0 = blockIdx.x * (int64_t)BLOCK; v0 < n; v0 += (int64_t)gridDim.x * BLOCK) {   // block-uniform
        const int64_t v = v0 + threadIdx.x;
        const bool hot = v < n && (double)indeg[v] >= thr;
        const uint64_t m = __ballot(hot);
        if (m == 0) continue;
        const int ln = __lane_id();
        unsigned int base = 0;
        if (ln == 0) base = atomicAdd(count, (unsigned int)__popcll(m));
        base = __shfl(base, 0);
        if (hot)
            keys[base + __popcll(m & ((1ull << ln) - 1ull))] = (uint64_t)(0xFFFFFFFFu - (uint32_t)indeg[v]) << 32 | (uint32_t)v;
    }
}

// Initial labels: 0 for a high-degree node (its search, hot[v] + 1, starts at
// it and none passes through it), H + 1 + v for any other node v.
__global__ void __launch_bounds__(BLOCK) k_order_init(int64_t n, uint32_t H, uint32_t *lab, int32_t *lev, uint64_t *claim) {
    for (int64_t v = blockIdx.x * (int64_t)BLOCK + threadIdx.x; v < n; v += (int64_t)gridDim.x * BLOCK) {
        lab[v] = H + 1 + (uint32_t)v;
        lev[v] = -1;
        claim[v] = ~0ull;
    }
}
__global__ void __launch_bounds__(BLOCK) k_hot_init(const uint64_t *keys, uint32_t H, uint32_t *lab, int32_t *lev,
                                                    uint32_t *disc, int32_t *perm) {
    for (uint32_t i = blockIdx.x * BLOCK + threadIdx.x; i < H; i += gridDim.x * BLOCK) {
        const uint32_t v = (uint32_t)keys[i];
        lab[v] = 0;
        lev[v] = 0;
        disc[v] = i;
        perm[v] = (int32_t)i;
    }
}

// The label a node passes on.
__device__ __forceinline__ uint32_t label_of(const uint32_t *lab, const uint32_t *disc, uint32_t u) {
    const uint32_t l = lab[u];
    return l ? l : disc[u] + 1;   // a high-degree node: its place among them
}

// One pass over the arcs: every successor takes the smaller label.
__global__ void __launch_bounds__(BLOCK) k_label_step(const uint64_t *keys, int64_t count, int shift, uint64_t mask,
                                                      uint32_t *lab, const uint32_t *disc, unsigned int *changed) {
    unsigned int c = 0;
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
        const uint64_t k = keys[i];
        const uint32_t lu = label_of(lab, disc, (uint32_t)(k >> shift));
        uint32_t *lv = &lab[k & mask];
        if (lu < *lv && atomicMin(lv, lu) > lu) ++c;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (__lane_id() == 0 && c) atomicAdd(changed, c);
}

// Level 0: the nodes no smaller label reached; they are found in input order.
__global__ void __launch_bounds__(BLOCK) k_roots(int64_t n, uint32_t H, const uint32_t *lab, int32_t *lev, uint32_t *disc) {
    for (int64_t v = blockIdx.x * (int64_t)BLOCK + threadIdx.x; v < n; v += (int64_t)gridDim.x * BLOCK)
        if (lab[v] == H + 1 + (uint32_t)v) {
            lev[v] = 0;
            disc[v] = (uint32_t)v;
        }
}

// Arcs out of level L into nodes of the same search not found yet: the first
// in queue order (the tail's discovery, then the place in its list) claims.
__global__ void __launch_bounds__(BLOCK) k_claim(const uint64_t *keys, int64_t count, int shift, uint64_t mask, int L,
                                                 const uint32_t *lab, const int32_t *lev, const uint32_t *disc,
                                                 uint64_t *claim) {
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
        const uint64_t k = keys[i];
        const uint32_t u = (uint32_t)(k >> shift);
        if (lev[u] != L) continue;
        const uint32_t v = (uint32_t)(k & mask);
        if (lev[v] >= 0 || lab[v] != label_of(lab, disc, u)) continue;
        const unsigned long long key = (unsigned long long)disc[u] << 32 | (uint32_t)i;
        if (key < claim[v]) atomicMin((unsigned long long *)&claim[v], key);
    }
}

// The nodes claimed in this level, unordered.
__global__ void __launch_bounds__(BLOCK) k_claimed(int64_t n, const int32_t *lev, const uint64_t *claim, uint64_t *keys,
                                                   uint32_t *ids, unsigned int *count) {
    for (int64_t v0 = blockIdx.x * (int64_t)BLOCK; v0 < n; v0 += (int64_t)gridDim.x * BLOCK) {   // block-uniform
        const int64_t v = v0 + threadIdx.x;
        const bool in = v < n && lev[v] < 0 && claim[v] != ~0ull;
        const uint64_t m = __ballot(in);
        if (m == 0) continue;
        const int ln = __lane_id();
        unsigned int base = 0;
        if (ln == 0) base = atomicAdd(count, (unsigned int)__popcll(m));
        base = __shfl(base, 0);
        if (in) {
            const unsigned int at = base + (unsigned int)__popcll(m & ((1ull << ln) - 1ull));
            keys[at] = claim[v];
            ids[at] = (uint32_t)v;
        }
    }
}
__global__ void __launch_bounds__(BLOCK) k_found(const uint32_t *ids, unsigned int count, int level, uint32_t first,
                                                 int32_t *lev, uint32_t *disc) {
    for (unsigned int i = blockIdx.x * BLOCK + threadIdx.x; i < count; i += gridDim.x * BLOCK) {
        lev[ids[i]] = level;
        disc[ids[i]] = first + i;
    }
}

// Sort keys of the final order (search, then discovery; a high-degree node last)
// and the numbers they give.
__global__ void __launch_bounds__(BLOCK) k_final_keys(int64_t n, const uint32_t *lab, const uint32_t *disc, uint64_t *keys,
                                                      uint32_t *ids) {
    for (int64_t v = blockIdx.x * (int64_t)BLOCK + threadIdx.x; v < n; v += (int64_t)gridDim.x * BLOCK) {
        keys[v] = lab[v] ? (uint64_t)lab[v] << 32 | disc[v] : ~0ull;
        ids[v] = (uint32_t)v;
    }
}
__global__ void __launch_bounds__(BLOCK) k_final_perm(const uint32_t *ids, int64_t count, uint32_t H, int32_t *perm) {
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK)
        perm[ids[i]] = (int32_t)(H + i);
}

// Relabel (perm: stored id of input node) and / or swap the halves.
__global__ void __launch_bounds__(BLOCK) k_rekey(const uint64_t *in, int64_t count, int shift, const int32_t *perm,
                                                 bool swap, uint64_t *out) {
    const uint64_t mask = (1ull << shift) - 1ull;
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
        uint64_t r = in[i] >> shift, c = in[i] & mask;
        if (perm) {
            r = (uint32_t)perm[r];
            c = (uint32_t)perm[c];
        }
        out[i] = swap ? (c << shift | r) : (r << shift | c);
    }
}

__global__ void k_fill_u64(unsigned long long *p, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__global__ void k_fill_i32z(int32_t *p, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

int grid_for(int64_t count) {
    const int64_t b = (count + BLOCK - 1) / BLOCK;
    return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

int bits_for(int64_t n) {
    int s = 1;
    while (s < 31 && (int64_t(1) << s) <= n) ++s;
    return s;
}

// A device block that goes back to the allocator when it leaves scope.
template <typename T> struct DevBuf {
    T *p = nullptr;
    bool get(int64_t count) {
        p = (T *)dev_malloc(sizeof(T) * (size_t)(count > 0 ? count : 1));
        return p != nullptr;
    }
    T *release() {
        T *q = p;
        p = nullptr;
        return q;
    }
    ~DevBuf() {
        if (p) dev_release(p);
    }
};

// `code`, once the stream is idle: an early way out gives blocks back (DevBuf)
// that queued work may still use.
int drained(hipStream_t st, int code) {
    (void)hipStreamSynchronize(st);
    return code;
}

#define BUILD_TRY(expr)                                                                                    \
    do {                                                                                                   \
        hipError_t e_ = (expr);                                                                            \
        if (e_ != hipSuccess)                                                                              \
            return drained(st, set_error(PP_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)));             \
    } while (0)

// keys[0, count) sorted into out (begin..end bits), with temporary storage.
int sort_keys(uint64_t *in, uint64_t *out, int64_t count, int bits, hipStream_t st) {
    size_t bytes = 0;
    BUILD_TRY(rocprim::radix_sort_keys(nullptr, bytes, in, out, (size_t)count, 0u, (unsigned)bits, st));
    DevBuf<unsigned char> tmp;
    if (!tmp.get((int64_t)bytes)) return drained(st, set_error(PP_ENOMEM, "radix sort storage of %zu bytes", bytes));
    BUILD_TRY(rocprim::radix_sort_keys(tmp.p, bytes, in, out, (size_t)count, 0u, (unsigned)bits, st));
    BUILD_TRY(hipStreamSynchronize(st));   // the storage goes back after the sort
    return PP_OK;
}

int sort_cols(uint32_t *in, uint32_t *out, int64_t count, int bits, hipStream_t st) {
    size_t bytes = 0;
    BUILD_TRY(rocprim::radix_sort_keys(nullptr, bytes, in, out, (size_t)count, 0u, (unsigned)bits, st));
    DevBuf<unsigned char> tmp;
    if (!tmp.get((int64_t)bytes)) return drained(st, set_error(PP_ENOMEM, "radix sort storage of %zu bytes", bytes));
    BUILD_TRY(rocprim::radix_sort_keys(tmp.p, bytes, in, out, (size_t)count, 0u, (unsigned)bits, st));
    BUILD_TRY(hipStreamSynchronize(st));
    return PP_OK;
}

// Pairs sorted by key (in place of the caller's second buffers).
int sort_pairs(uint64_t *k_in, uint64_t *k_out, uint32_t *v_in, uint32_t *v_out, int64_t count, hipStream_t st) {
    size_t bytes = 0;
    BUILD_TRY(rocprim::radix_sort_pairs(nullptr, bytes, k_in, k_out, v_in, v_out, (size_t)count, 0u, 64u, st));
    DevBuf<unsigned char> tmp;
    if (!tmp.get((int64_t)bytes)) return drained(st, set_error(PP_ENOMEM, "radix sort storage of %zu bytes", bytes));
    BUILD_TRY(rocprim::radix_sort_pairs(tmp.p, bytes, k_in, k_out, v_in, v_out, (size_t)count, 0u, 64u, st));
    BUILD_TRY(hipStreamSynchronize(st));
    return PP_OK;
}

// The storage order of one graph with high-degree nodes, as pp_csr_build's host
// searches number it: those nodes first, by decreasing in-degree, then the
// others in the order breadth-first searches find them, started at each
// high-degree node and then at each node not yet found, in input order.  keys:
// the arcs, sorted, by input id; indeg: in-degrees.  *done stays false when the
// searches are too deep for passes over all arcs (or there is no high-degree
// node, or no memory): the host searches them then.
// The search that finds a node is the first that reaches it over nodes that are
// not high-degree ones, whichever nodes earlier searches took on the way (they
// would have found it too): the least label over the arcs.  Within a search the
// queue holds a level's nodes by their first tail's place in the queue, then by
// the place in that tail's list: the least such key claims a node, and a sort
// of each level's claims gives the discovery numbers of the next.
// Whole builds, pairs on the device: R-MAT 17 7.0 -> 3.1 ms, R-MAT 20 77 -> 14 ms,
// R-MAT 24 2.10 -> 0.25 s, undirected R-MAT 18 42 -> 5.7 ms.
constexpr int ORDER_PASSES = 32, ORDER_LEVELS = 64;
int device_order(const uint64_t *keys, int64_t count, int64_t n, int shift, const int32_t *indeg, double thr,
                 std::vector<int32_t> &perm, DevBuf<int32_t> &perm_d, bool *done, hipStream_t st) {
    *done = false;
    const uint64_t mask = (1ull << shift) - 1ull;
    DevBuf<uint32_t> lab, disc, i0, i1;
    DevBuf<int32_t> lev, pd;
    DevBuf<uint64_t> claim, s0, s1;
    DevBuf<unsigned int> cnt;
    if (!cnt.get(1) || !s0.get(n) || !s1.get(n) || !pd.get(n) || !lab.get(n) || !disc.get(n) || !lev.get(n) ||
        !claim.get(n) || !i0.get(n) || !i1.get(n))
        return drained(st, PP_OK);   // the host's searches need no device memory
    auto zero = [&]() { hipLaunchKernelGGL(k_fill_i32z, dim3(1), dim3(BLOCK), 0, st, (int32_t *)cnt.p, (int64_t)1); };
    auto read = [&](unsigned int &c) -> int {
        BUILD_TRY(hipGetLastError());
        BUILD_TRY(hipMemcpyAsync(&c, cnt.p, sizeof(c), hipMemcpyDeviceToHost, st));
        BUILD_TRY(hipStreamSynchronize(st));
        return PP_OK;
    };
    int rc;
    unsigned int H = 0, c = 0;
    zero();
    hipLaunchKernelGGL(k_hot_keys, dim3(grid_for(n)), dim3(BLOCK), 0, st, indeg, n, thr, s0.p, cnt.p);
    if ((rc = read(H))) return rc;
    if (H == 0) return PP_OK;   // lattices, paths: many levels
    if ((rc = sort_keys(s0.p, s1.p, H, 64, st))) return rc == PP_ENOMEM ? PP_OK : rc;
    hipLaunchKernelGGL(k_order_init, dim3(grid_for(n)), dim3(BLOCK), 0, st, n, H, lab.p, lev.p, claim.p);
    hipLaunchKernelGGL(k_hot_init, dim3(grid_for(H)), dim3(BLOCK), 0, st, s1.p, H, lab.p, lev.p, disc.p, pd.p);
    for (int pass = 1;; ++pass) {
        // a look at the passes' changes from the fourth on: while an eighth of the
        // nodes still change, the labels travel too far
        const bool look = pass >= 4;
        if (look) zero();
        hipLaunchKernelGGL(k_label_step, dim3(grid_for(count)), dim3(BLOCK), 0, st, keys, count, shift, mask, lab.p,
                           disc.p, cnt.p);
        if (!look) continue;
        if ((rc = read(c))) return rc;
        if (c == 0) break;
        if (pass >= ORDER_PASSES || (int64_t)c * 8 > n) return PP_OK;
    }
    hipLaunchKernelGGL(k_roots, dim3(grid_for(n)), dim3(BLOCK), 0, st, n, H, lab.p, lev.p, disc.p);
    uint32_t first = (uint32_t)n;   // discovery numbers: roots by id, then the levels' nodes
    for (int L = 0;; ++L) {
        zero();
        hipLaunchKernelGGL(k_claim, dim3(grid_for(count)), dim3(BLOCK), 0, st, keys, count, shift, mask, L, lab.p, lev.p,
                           disc.p, claim.p);
        hipLaunchKernelGGL(k_claimed, dim3(grid_for(n)), dim3(BLOCK), 0, st, n, lev.p, claim.p, s0.p, i0.p, cnt.p);
        if ((rc = read(c))) return rc;
        if (c == 0) break;
        if (L == ORDER_LEVELS) return PP_OK;   // the stream is idle here: read() has waited
        if ((rc = sort_pairs(s0.p, s1.p, i0.p, i1.p, c, st))) return rc == PP_ENOMEM ? PP_OK : rc;
        hipLaunchKernelGGL(k_found, dim3(grid_for(c)), dim3(BLOCK), 0, st, i1.p, c, L + 1, first, lev.p, disc.p);
        first += c;
    }
    hipLaunchKernelGGL(k_final_keys, dim3(grid_for(n)), dim3(BLOCK), 0, st, n, lab.p, disc.p, s0.p, i0.p);
    BUILD_TRY(hipGetLastError());
    if ((rc = sort_pairs(s0.p, s1.p, i0.p, i1.p, n, st))) return rc == PP_ENOMEM ? PP_OK : rc;
    perm.resize((size_t)n);   // (may throw: the stream is idle)
    hipLaunchKernelGGL(k_final_perm, dim3(grid_for(n - H)), dim3(BLOCK), 0, st, i1.p, n - (int64_t)H, H, pd.p);
    BUILD_TRY(hipGetLastError());
    BUILD_TRY(hipMemcpyAsync(perm.data(), pd.p, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, st));
    BUILD_TRY(hipStreamSynchronize(st));
    perm_d.p = pd.release();
    *done = true;
    return PP_OK;
}

// Rows of n nodes from count sorted keys (no duplicates): offsets and columns.
int keys_to_rows(const uint64_t *keys, int64_t count, int64_t n, int shift, DevRows &out, hipStream_t st) {
    DevBuf<unsigned long long> len;
    DevBuf<int64_t> rp;
    DevBuf<int32_t> col;
    if (!len.get(n + 1) || !rp.get(n + 1) || !col.get(count))
        return drained(st, set_error(PP_ENOMEM, "device rows of %lld nodes and %lld arcs", (long long)n, (long long)count));
    hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(n + 1)), dim3(BLOCK), 0, st, len.p, n + 1);
    if (count > 0) {
        hipLaunchKernelGGL(k_row_lengths, dim3(grid_for(count)), dim3(BLOCK), 0, st, keys, count, shift, len.p);
        hipLaunchKernelGGL(k_key_cols, dim3(grid_for(count)), dim3(BLOCK), 0, st, keys, count, (1ull << shift) - 1ull,
                           col.p);
    }
    BUILD_TRY(hipGetLastError());
    size_t bytes = 0;
    const int64_t *lin = reinterpret_cast<const int64_t *>(len.p);
    BUILD_TRY(rocprim::exclusive_scan(nullptr, bytes, lin, rp.p, (int64_t)0, (size_t)(n + 1), rocprim::plus<int64_t>(), st));
    DevBuf<unsigned char> tmp;
    if (!tmp.get((int64_t)bytes)) return drained(st, set_error(PP_ENOMEM, "scan storage of %zu bytes", bytes));
    BUILD_TRY(rocprim::exclusive_scan(tmp.p, bytes, lin, rp.p, (int64_t)0, (size_t)(n + 1), rocprim::plus<int64_t>(), st));
    BUILD_TRY(hipStreamSynchronize(st));
    out.rp = rp.release();
    out.col = col.release();
    out.m = count;
    return PP_OK;
}

}  // namespace

int device_check_arcs(const int32_t *a, const int32_t *b, int64_t m, int64_t n, const int32_t *node_graph,
                      int64_t *first_bad, hipStream_t st) {
    *first_bad = -1;
    if (m <= 0) return PP_OK;
    DevBuf<unsigned long long> flag;
    if (!flag.get(1)) return drained(st, set_error(PP_ENOMEM, "a flag"));
    const unsigned long long none = ~0ull;
    BUILD_TRY(hipMemcpyAsync(flag.p, &none, sizeof(none), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_check_arcs, dim3(grid_for(m)), dim3(BLOCK), 0, st, a, b, m, n, node_graph, flag.p);
    BUILD_TRY(hipGetLastError());
    unsigned long long got = 0;
    BUILD_TRY(hipMemcpyAsync(&got, flag.p, sizeof(got), hipMemcpyDeviceToHost, st));
    BUILD_TRY(hipStreamSynchronize(st));
    *first_bad = got == none ? -1 : (int64_t)got;
    return PP_OK;
}

int device_build(int64_t n, int64_t m, const int32_t *a, const int32_t *b, bool undirected, const OrderFn &order,
                 bool searches, DevRows &rows, DevRows &trows, std::vector<int32_t> &perm, hipStream_t st) {
    const int shift = bits_for(n);
    const int bits = 2 * shift;
    const uint64_t mask = (1ull << shift) - 1ull;
    const uint64_t no_arc = (1ull << bits) - 1ull;
    const int64_t slots = undirected ? 2 * m : m;
    if (slots >= (int64_t(1) << 32))
        return set_error(PP_EINVAL, "%lld arc keys: the device build takes fewer than 2^32 (PP_BUILD_ON_HOST)",
                         (long long)slots);
    // sorted keys without self-loops and duplicates
    DevBuf<uint64_t> k0, k1;
    if (!k0.get(slots) || !k1.get(slots)) return drained(st, set_error(PP_ENOMEM, "%lld arc keys", (long long)slots));
    int64_t count = 0;
    if (m > 0) {
        hipLaunchKernelGGL(k_arc_keys, dim3(grid_for(m)), dim3(BLOCK), 0, st, a, b, m, shift, undirected, no_arc,
                           k0.p);
        BUILD_TRY(hipGetLastError());
        int rc = sort_keys(k0.p, k1.p, slots, bits, st);
        if (rc) return rc;
        DevBuf<unsigned int> ucount;
        if (!ucount.get(1)) return drained(st, set_error(PP_ENOMEM, "a count"));
        size_t bytes = 0;
        BUILD_TRY(rocprim::unique(nullptr, bytes, k1.p, k0.p, ucount.p, (size_t)slots, rocprim::equal_to<uint64_t>(), st));
        DevBuf<unsigned char> tmp;
        if (!tmp.get((int64_t)bytes)) return drained(st, set_error(PP_ENOMEM, "unique storage of %zu bytes", bytes));
        BUILD_TRY(rocprim::unique(tmp.p, bytes, k1.p, k0.p, ucount.p, (size_t)slots, rocprim::equal_to<uint64_t>(), st));
        unsigned int u = 0;
        BUILD_TRY(hipMemcpyAsync(&u, ucount.p, sizeof(u), hipMemcpyDeviceToHost, st));
        BUILD_TRY(hipStreamSynchronize(st));
        count = (int64_t)u;
        if (count > 0) {
            uint64_t last = 0;
            BUILD_TRY(hipMemcpyAsync(&last, k0.p + (count - 1), sizeof(last), hipMemcpyDeviceToHost, st));
            BUILD_TRY(hipStreamSynchronize(st));
            if (last == no_arc) --count;
        }
    }
    // k0[0, count): the stored arcs by input id, sorted by row then column.
    // Degrees for the storage order: out-degrees from the rows, in-degrees by column.
    DevBuf<int32_t> perm_d;
    {
        DevRows r0;
        int rc = keys_to_rows(k0.p, count, n, shift, r0, st);
        if (rc) return rc;
        DevBuf<int64_t> rp0;
        DevBuf<int32_t> col0;
        rp0.p = r0.rp;
        col0.p = r0.col;
        DevBuf<int32_t> indeg;
        if (!indeg.get(n)) return drained(st, set_error(PP_ENOMEM, "in-degrees of %lld nodes", (long long)n));
        hipLaunchKernelGGL(k_fill_i32z, dim3(grid_for(n)), dim3(BLOCK), 0, st, indeg.p, n);
        if (count > 0) {
            // the columns alone, sorted, in the key buffer free now: an atomic per
            // run end instead of one per arc (R-MAT 24: 23.9 ms of atomics, 4.5 ms
            // for the sort and the runs; R-MAT 17: 0.31 ms, 0.07 ms)
            uint32_t *c0 = reinterpret_cast<uint32_t *>(k1.p), *c1 = c0 + count;
            hipLaunchKernelGGL(k_key_cols, dim3(grid_for(count)), dim3(BLOCK), 0, st, k0.p, count, mask,
                               reinterpret_cast<int32_t *>(c0));
            BUILD_TRY(hipGetLastError());
            rc = sort_cols(c0, c1, count, shift, st);
            if (rc && rc != PP_ENOMEM) return rc;
            if (rc) hipLaunchKernelGGL(k_col_adds, dim3(grid_for(count)), dim3(BLOCK), 0, st, c0, count, indeg.p);
            else hipLaunchKernelGGL(k_col_counts, dim3(grid_for(count)), dim3(BLOCK), 0, st, c1, count, indeg.p);
        }
        BUILD_TRY(hipGetLastError());
        bool moved = false, done = false;
        if (searches && count > 0) {
            // the host's threshold: max(8, twice the mean in-degree)
            const double mean = (double)count / (double)n;
            rc = device_order(k0.p, count, n, shift, indeg.p, mean * 2.0 > 8.0 ? mean * 2.0 : 8.0, perm, perm_d, &done, st);
            if (rc) return rc;
            for (int64_t x = 0; done && x < n && !moved; ++x) moved = perm[(size_t)x] != (int32_t)x;
        }
        std::vector<int64_t> rp_h, trp_h;
        std::vector<int32_t> deg_h;
        if (!done) {
            BUILD_TRY(hipStreamSynchronize(st));   // the vectors may throw
            rp_h.resize((size_t)n + 1);
            trp_h.assign((size_t)n + 1, 0);
            deg_h.resize((size_t)n);
            BUILD_TRY(hipMemcpyAsync(rp_h.data(), rp0.p, sizeof(int64_t) * (size_t)(n + 1), hipMemcpyDeviceToHost, st));
            BUILD_TRY(hipMemcpyAsync(deg_h.data(), indeg.p, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, st));
            BUILD_TRY(hipStreamSynchronize(st));
            for (int64_t v = 0; v < n; ++v) trp_h[(size_t)v + 1] = trp_h[(size_t)v] + deg_h[(size_t)v];
        }
        std::vector<int32_t> col_h;
        hipError_t col_err = hipSuccess;
        const std::function<const int32_t *()> col = [&]() -> const int32_t * {
            if (col_h.empty() && count > 0) {
                col_h.resize((size_t)count);
                col_err = hipMemcpyAsync(col_h.data(), col0.p, sizeof(int32_t) * (size_t)count, hipMemcpyDeviceToHost, st);
                if (col_err == hipSuccess) col_err = hipStreamSynchronize(st);
            }
            return col_h.data();
        };
        if (!done) moved = order(rp_h, trp_h, col, perm);
        BUILD_TRY(col_err);
        if (!moved) {
            perm.clear();
            rows.rp = rp0.release();
            rows.col = col0.release();
            rows.m = count;
        }
    }
    if (!perm.empty()) {
        if (!perm_d.p) {
            if (!perm_d.get(n)) return drained(st, set_error(PP_ENOMEM, "the storage order"));
            BUILD_TRY(hipMemcpyAsync(perm_d.p, perm.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, st));
        }
        // rows in storage order: relabel, sort
        if (count > 0) {
            hipLaunchKernelGGL(k_rekey, dim3(grid_for(count)), dim3(BLOCK), 0, st, k0.p, count, shift, perm_d.p, false,
                               k1.p);
            BUILD_TRY(hipGetLastError());
            int rc = sort_keys(k1.p, k0.p, count, bits, st);
            if (rc) return rc;
        }
        int rc = keys_to_rows(k0.p, count, n, shift, rows, st);
        if (rc) return rc;
    }
    // the transpose: the (relabelled) keys with the halves swapped, sorted
    if (count > 0) {
        hipLaunchKernelGGL(k_rekey, dim3(grid_for(count)), dim3(BLOCK), 0, st, k0.p, count, shift, nullptr, true, k1.p);
        BUILD_TRY(hipGetLastError());
        int rc = sort_keys(k1.p, k0.p, count, bits, st);
        if (rc) return rc;
    }
    return keys_to_rows(k0.p, count, n, shift, trows, st);
}

}  // namespace pp
