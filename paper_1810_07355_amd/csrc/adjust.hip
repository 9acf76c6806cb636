// Graph adjustment on the GPU:
//   static degree adjustment, ConstructAdjustedGraph (Algorithm 2),
//   the same with constraints, ConstructAdjustedGraphWithConstraint
//   (Algorithm 3), and path adjustment, AdjustPath with HasPath (Algorithms 4 and 5).
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <cstdint>
#include <vector>

#include "onng_internal.h"
#include "wave.h"

namespace onng {

namespace {

template <typename LenT>
__device__ __forceinline__ uint32_t len_ord(LenT v) {
    if constexpr (std::is_integral<LenT>::value) return (uint32_t)v;   // int32 lengths
    else return ord_f32((float)v);
}

// ------------------------------------------------------------ Algorithm 2 --
// Row o of the kNN table gives, in order, the edges S of Algorithm 2.  With the
// loop guard "p <= e_o or p <= e_i", step p of node o adds o -> n (p <= e_o) and
// n -> o (p <= e_i).  As sets: N(o) = F(o) u Rv(o), F(o) = first e_o of row o,
// Rv(o) = {m : o among the first e_i of row m}.  An edge present in both
// ways is inserted once, by whichever step comes first in the loop (node
// ascending, then p): the reverse copy when the far end has the smaller id,
// and it keeps that copy's length.

// Every reverse candidate (o, m) goes to o's segment first, m's forward edges
// are its own row, and one wave per node then drops the reverse copies of its
// forward edges.  Whether m -> o repeats a forward edge of o is thus decided
// next to both lists; looked up instead in row o for every candidate, twice
// (count, then scatter), one lane per row, it was 17 of the 19 ms that
// 200,003 rows of 100 took (e_o = 20, e_i = 60; now 1.06 ms, of which the
// scattered 8-byte keys are 0.23 and the merge 0.25).

__device__ __forceinline__ int row_len(const int32_t *row, int k) {
    int l = 0;
    while (l < k && row[l] >= 0) l++;
    return l;
}

// Node of a wave: blocks go to the 8 XCDs in turn, so each XCD takes one run of
// consecutive nodes, whose rows share neighbours (and so segment lines).
__device__ __forceinline__ int64_t xcd_node(int64_t n) {
    const int64_t nblk = gridDim.x, per = nblk / 8, rest = nblk - per * 8;
    const int64_t xcd = blockIdx.x % 8, at = blockIdx.x / 8;
    const int64_t v = (xcd * per + min(xcd, rest) + at) * (blockDim.x / WAVE) + uni(threadIdx.x / WAVE);
    return v < n ? v : -1;
}

// Row m (first max(eo, ei) entries, up to its padding): its forward count, and
// for each reverse candidate its place among those of the target.  A block
// takes SA_ROWS consecutive rows, which share targets (the rows are in
// locality order): it counts them per target in a hash table in LDS and asks
// the target's global counter for one range per block.  One global atomic per
// candidate ran at 21G a second, 0.58 ms for 12M candidates; per block and
// target, 0.26 ms.
constexpr int SA_WAVES = 8, SA_RPW = 16, SA_ROWS = SA_WAVES * SA_RPW;   // rows per wave, block
// Slots of the table: neighbouring rows share most targets.  A target that
// finds no place within SA_PROBES slots (unordered rows: up to 8192 distinct
// ones) goes to the global counter directly.
constexpr int SA_HASH = 4096, SA_PROBES = 8;

__global__ void __launch_bounds__(SA_WAVES * WAVE) sa_count_kernel(const int32_t *knn, int64_t n,
                                                                   int k, int eo, int ei,
                                                                   int32_t *rcnt, int32_t *slot,
                                                                   int32_t *fcnt) {
    __shared__ int32_t hid[SA_HASH];   // target, -1 empty
    __shared__ int32_t hcnt[SA_HASH];  // its candidates in this block, then its range's start
    const int lane = lane_id();
    const int64_t m0 = (int64_t)blockIdx.x * SA_ROWS + uni(threadIdx.x / WAVE) * SA_RPW;
    const int lim = max(eo, ei);
    int len[SA_RPW];
#pragma unroll
    for (int r = 0; r < SA_RPW; r++) len[r] = m0 + r < n ? lim : 0;
    for (int t0 = 0; t0 < lim; t0 += WAVE) {
        __syncthreads();
        for (int i = threadIdx.x; i < SA_HASH; i += blockDim.x) hid[i] = -1, hcnt[i] = 0;
        __syncthreads();
        // per row: this lane's table place (low 16 bits) and its candidate's
        // number among the block's of that target
        uint32_t at[SA_RPW];
#pragma unroll
        for (int r = 0; r < SA_RPW; r++) {
            const int t = t0 + lane;
            const int32_t o = t < len[r] ? knn[(m0 + r) * k + t] : 0;
            const uint64_t pad = ballot(o < 0);
            if (pad) len[r] = t0 + (int)__builtin_ctzll(pad);
            at[r] = ~0u;
            if (t < min(ei, len[r]) && o < n) {
                uint32_t h = ((uint32_t)o * 2654435761u) >> (32 - __builtin_ctz(SA_HASH));
                int p = 0;
                for (int32_t was; p < SA_PROBES && (was = atomicCAS(&hid[h], -1, o)) != -1 && was != o; p++)
                    h = (h + 1) & (SA_HASH - 1);
                if (p < SA_PROBES) at[r] = h | (uint32_t)atomicAdd(&hcnt[h], 1) << 16;
                else slot[(m0 + r) * ei + t] = atomicAdd(&rcnt[o], 1);
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < SA_HASH; i += blockDim.x)
            if (hid[i] >= 0) hcnt[i] = atomicAdd(&rcnt[hid[i]], hcnt[i]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < SA_RPW; r++)
            if (at[r] != ~0u)
                slot[(m0 + r) * ei + t0 + lane] = hcnt[at[r] & 0xFFFFu] + (int32_t)(at[r] >> 16);
    }
#pragma unroll
    for (int r = 0; r < SA_RPW; r++)
        if (lane == r && m0 + r < n) fcnt[m0 + r] = min(eo, len[r]);
}

// segment sizes: reverse candidates and forward edges
__global__ void sa_sizes_kernel(const int32_t *rcnt, const int32_t *fcnt, int64_t n, int64_t *size) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v <= n) size[v] = v < n ? (int64_t)rcnt[v] + fcnt[v] : 0;
}

template <typename LenT>
__global__ void __launch_bounds__(256) sa_scatter_kernel(const int32_t *knn, const LenT *kd, int64_t n,
                                                         int k, int ei, const int64_t *seg,
                                                         const int32_t *slot, uint64_t *keys) {
    const int64_t m = xcd_node(n);
    if (m < 0) return;
    const int lane = lane_id();
    const int32_t *row = knn + m * k;
    int len = ei;
    for (int t0 = 0; t0 < len; t0 += WAVE) {
        const int t = t0 + lane;
        const int32_t o = t < ei ? row[t] : 0;
        const uint64_t pad = ballot(o < 0);
        if (pad) len = t0 + (int)__builtin_ctzll(pad);
        if (t < len && o < n)
            keys[seg[o] + slot[m * ei + t]] = make_key(len_ord(kd[m * k + t]), (uint32_t)m);
    }
}

// Node o's segment: reverse candidates whose id is a forward edge of o go, the
// forward edges follow the rest (unsorted), and cnt[o] is what remains.  A
// forward edge to a smaller id takes the dropped copy's length.
template <typename LenT>
__global__ void __launch_bounds__(256) sa_merge_kernel(const int32_t *knn, const LenT *kd, int64_t n,
                                                       int k, const int32_t *rcnt,
                                                       const int32_t *fcnt, const int64_t *seg,
                                                       uint64_t *keys, int64_t *cnt) {
    const int64_t o = xcd_node(n);
    if (o < 0) return;
    const int lane = lane_id();
    uint64_t *s = keys + seg[o];
    const int f = uni(fcnt[o]), r0 = uni(rcnt[o]);
    int r = r0;
    for (int f0 = 0; f0 < f; f0 += WAVE) {
        const int fn = min(WAVE, f - f0);
        int32_t id = 0;
        uint64_t fkey = 0;
        if (lane < fn) {
            id = knn[o * k + f0 + lane];
            fkey = make_key(len_ord(kd[o * k + f0 + lane]), (uint32_t)id);
        }
        int kept = 0;
        for (int c0 = 0; c0 < r; c0 += WAVE) {
            const bool has = c0 + lane < r;
            const uint64_t key = has ? s[c0 + lane] : 0;
            const uint32_t rid = (uint32_t)key;
            bool drop = false;
            for (int e = 0; e < fn; e++) {
                const uint32_t fid = (uint32_t)__builtin_amdgcn_readlane(id, e);
                const uint64_t hit = ballot(has && rid == fid);
                if (!hit) continue;
                drop = drop || ((hit >> lane) & 1);
                if ((int64_t)fid < o) {
                    const uint64_t rk = (uint64_t)readlane64((int64_t)key, (int)__builtin_ctzll(hit));
                    if (lane == e) fkey = rk;
                }
            }
            const uint64_t stay = ballot(has && !drop);
            if (has && !drop) s[kept + mbcnt(stay)] = key;   // at or before where it was read
            kept += __popcll(stay);
        }
        r = kept;
        if (lane < fn) s[r0 + f0 + lane] = fkey;
        // the next 64 forward edges read what other lanes moved
        if (f0 + WAVE < f) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    }
    if (r < r0)
        for (int c = lane; c < f; c += WAVE) {
            const uint64_t key = s[r0 + c];   // this lane's own store
            s[r + c] = key;
        }
    if (lane == 0) cnt[o] = r + f;
}

// Short rows (at most SA_SHORT entries count) of few nodes: a lane a row, which looks
// its own id up in the short row of each target, for the counts and again for the
// keys.  Three launches fewer than the way by segments, which such calls are bound
// by; us, so / by segments: 1000 nodes, e_o = e_i = 1: 65 / 104, 2 and 5: 77 / 105;
// 10,000 nodes, 1 and 3: 101 / 122.  The looking up costs e_o e_i per node: at 4000
// nodes, 5 and 5: 123 / 117, at 30,000, 2 and 5: 147 / 140.
constexpr int SA_SHORT = 5;

__device__ __forceinline__ bool in_row(const int32_t *row, int lim, int32_t x) {
    for (int t = 0; t < lim && row[t] >= 0; t++)
        if (row[t] == x) return true;
    return false;
}

__global__ void sa_short_count_kernel(const int32_t *knn, int64_t n, int k, int eo, int ei, int64_t *cnt) {
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    const int32_t *row = knn + m * k;
    const int len = row_len(row, max(eo, ei));
    atomicAdd((unsigned long long *)&cnt[m], (unsigned long long)min(eo, len));
    for (int t = 0; t < min(ei, len); t++)
        if (row[t] < n && !in_row(knn + (int64_t)row[t] * k, eo, (int32_t)m))
            atomicAdd((unsigned long long *)&cnt[row[t]], 1ull);
}

// forward edges first, then the reverse ones that are none of them
template <typename LenT>
__global__ void sa_short_scatter_kernel(const int32_t *knn, const LenT *kd, int64_t n, int k, int eo, int ei,
                                        const int64_t *off, int32_t *cursor, uint64_t *keys) {
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    const int32_t *row = knn + m * k;
    const int len = row_len(row, max(eo, ei));
    for (int t = 0; t < min(eo, len); t++) {
        const int64_t o = row[t];
        LenT l = kd[m * k + t];
        if (o < m)   // the copy that o's step adds comes first
            for (int u = 0; u < ei && knn[o * k + u] >= 0; u++)
                if (knn[o * k + u] == m) {
                    l = kd[o * k + u];
                    break;
                }
        keys[off[m] + t] = make_key(len_ord(l), (uint32_t)o);
    }
    for (int t = 0; t < min(ei, len); t++) {
        const int64_t o = row[t];
        if (o >= n || in_row(knn + o * k, eo, (int32_t)m)) continue;
        const int at = min(eo, row_len(knn + o * k, eo)) + atomicAdd(&cursor[o], 1);
        keys[off[o] + at] = make_key(len_ord(kd[m * k + t]), (uint32_t)m);
    }
}

// ------------------------------------------------------------ segment sort --
// List v: cnt = off[v+1] - off[v] keys at keys[seg[v]] to nbrs/lens at off[v],
// in ascending order; equal keys keep their order.  A key's place is the
// number of smaller ones: the list sits in LDS and every lane compares its
// keys with all of them, read two at a time by broadcast.  Lists of at most
// 256 take one wave (up to four keys a lane), four lists per block: the places
// of a list of m keys cost m / 2 broadcasts and 2 m / 64 compares a lane, less
// than a bitonic network's exchanges there.  Longer ones are queued for blocks
// of their own, which sort up to 4096 keys in LDS by a bitonic network.  Up to 1024
// lists in all go to such blocks directly, without a queue.
// (13.5M edges in 200,003 lists, 5,000 of them long: 0.15 + 0.10 ms; the long
// ones by counting 0.70 ms; one block of 256 threads per list, every place
// counted, 2.0 ms.)

constexpr int SEG_WAVE = 256;      // longest list of one wave
constexpr int SEG_LDS = 4096;      // longest list held in LDS
constexpr int SEG_BLOCKS = 1024;   // blocks that drain the queue of long lists

template <typename LenT>
__device__ __forceinline__ void seg_put(int32_t *nbrs, LenT *lens, int64_t at, uint64_t key) {
    nbrs[at] = (int32_t)(uint32_t)key;
    const uint32_t d = (uint32_t)(key >> 32);
    if constexpr (std::is_integral<LenT>::value) lens[at] = (LenT)d;
    else lens[at] = unord_f32(d);
}

// rank of R keys per lane (index p * 64 + lane) among the m keys of `sk`;
// TIES: equal keys in index order
template <int R, bool TIES>
__device__ __forceinline__ void seg_ranks(const uint64_t *sk, int m, const uint64_t (&key)[R],
                                          int (&rank)[R]) {
    const int lane = lane_id();
#pragma unroll
    for (int p = 0; p < R; p++) rank[p] = 0;
    for (int j = 0; j < m; j += 2) {   // sk[m] pads an odd count
        const ulonglong2 o = *reinterpret_cast<const ulonglong2 *>(sk + j);
#pragma unroll
        for (int p = 0; p < R; p++) {
            rank[p] += (uint64_t)o.x < key[p];
            rank[p] += (uint64_t)o.y < key[p];
            if (TIES) {
                rank[p] += (uint64_t)o.x == key[p] && j < p * WAVE + lane;
                rank[p] += (uint64_t)o.y == key[p] && j + 1 < p * WAVE + lane;
            }
        }
    }
}

template <typename LenT, int R>
__device__ __forceinline__ void seg_sort_wave(const uint64_t *src, uint64_t *sk, int m, int64_t b,
                                              int32_t *nbrs, LenT *lens) {
    const int lane = lane_id();
    uint64_t key[R];
    int rank[R];
#pragma unroll
    for (int p = 0; p < R; p++) {
        const int i = p * WAVE + lane;
        key[p] = i < m ? src[i] : KEY_MAX;
        sk[i] = key[p];
    }
    if (lane == 0) sk[R * WAVE] = KEY_MAX;
    wave_sync();
    seg_ranks<R, false>(sk, m, key, rank);
    // without equal keys the ranks are 0 .. m-1; with some their sum is smaller
    int sum = 0;
#pragma unroll
    for (int p = 0; p < R; p++) sum += p * WAVE + lane < m ? rank[p] : 0;
    for (int s = 32; s >= 1; s >>= 1) sum += __shfl_xor(sum, s);
    if (uni(sum) != m * (m - 1) / 2) seg_ranks<R, true>(sk, m, key, rank);
#pragma unroll
    for (int p = 0; p < R; p++)
        if (p * WAVE + lane < m) seg_put(nbrs, lens, b + rank[p], key[p]);
}

template <typename LenT>
__global__ void __launch_bounds__(256) seg_sort_kernel(const int64_t *seg, const int64_t *off,
                                                       int64_t n, const uint64_t *keys,
                                                       int32_t *nbrs, LenT *lens, int32_t *queue,
                                                       int32_t *n_queue) {
    __shared__ __attribute__((aligned(16))) uint64_t sk_all[4][SEG_WAVE + 2];
    const int64_t v = xcd_node(n);
    if (v < 0) return;
    const int64_t b = off[v], m64 = off[v + 1] - b;
    if (m64 == 0) return;
    if (m64 > SEG_WAVE) {
        if (lane_id() == 0) queue[atomicAdd(n_queue, 1)] = (int32_t)v;
        return;
    }
    const int m = uni((int)m64);
    const uint64_t *src = keys + seg[v];
    uint64_t *sk = sk_all[threadIdx.x / WAVE];
    if (m <= 64) seg_sort_wave<LenT, 1>(src, sk, m, b, nbrs, lens);
    else if (m <= 128) seg_sort_wave<LenT, 2>(src, sk, m, b, nbrs, lens);
    else if (m <= 192) seg_sort_wave<LenT, 3>(src, sk, m, b, nbrs, lens);
    else seg_sort_wave<LenT, 4>(src, sk, m, b, nbrs, lens);
}

template <typename LenT>
__global__ void __launch_bounds__(512) seg_sort_long_kernel(const int64_t *seg, const int64_t *off,
                                                            const uint64_t *keys, int32_t *nbrs,
                                                            LenT *lens, const int32_t *queue,
                                                            const int32_t *n_queue, int n_lists) {
    __shared__ uint64_t sk[SEG_LDS];
    const int total = queue ? *n_queue : n_lists;
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int64_t v = queue ? queue[q] : q;
        const int64_t b = off[v], m = off[v + 1] - b;
        const uint64_t *src = keys + seg[v];
        __syncthreads();
        if (m <= SEG_LDS) {
            // bitonic sort over the next power of two (equal keys are equal
            // edges, so their order does not matter)
            const int w = pow2_at_least((int)m);
            for (int i = threadIdx.x; i < w; i += blockDim.x) sk[i] = i < m ? src[i] : KEY_MAX;
            for (int size = 2; size <= w; size <<= 1)
                for (int d = size >> 1; d > 0; d >>= 1) {
                    __syncthreads();
                    for (int t = threadIdx.x; t < w / 2; t += blockDim.x) {
                        const int i = 2 * t - (t & (d - 1));   // lower of the pair (i, i + d)
                        const uint64_t lo = sk[i], hi = sk[i + d];
                        if ((lo > hi) == ((i & size) == 0)) sk[i] = hi, sk[i + d] = lo;
                    }
                }
            __syncthreads();
            for (int i = threadIdx.x; i < m; i += blockDim.x) seg_put(nbrs, lens, b + i, sk[i]);
        } else {
            for (int64_t i = threadIdx.x; i < m; i += blockDim.x) {
                const uint64_t x = src[i];
                int64_t rank = 0;
                for (int64_t j = 0; j < m; j++) rank += src[j] < x || (src[j] == x && j < i);
                seg_put(nbrs, lens, b + rank, x);
            }
        }
    }
}

// ------------------------------------------------------------ Algorithm 3 --
// G_t = ConstructAdjustedGraph(G, 0, e_i): N(G_t, o) = {m : o among the first
// e_i of row m}, each edge with row m's length.  The first loop's in-degree
// bound never binds: only the (at most e_i) nodes of row n's head can add an
// edge into n, each of them considers n once, so whenever one does, fewer
// than e_i have added it before.  What remains decides every edge on its own:
// the first of row n's head in processing order (ascending (|N(G_t, x)|, x))
// meets n with in-degree 0 and adds it; any later one adds it only while its
// own out-degree is below e_o, i.e. for the first e_o members of N(G_t, o) in
// (length, id) order, all of which the loop keeps.  So o -> n is kept iff n is
// among those first e_o or o is n's first source.  The fill loop matters only
// for nodes with |N(G_t, o)| < e_o, whose first loop kept all of N(G_t, o): it
// appends the members of row o not already present, nearest first, up to e_o.

__global__ void sac_rcount_kernel(const int32_t *knn, int64_t n, int k, int ei, int64_t *cnt) {
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    const int32_t *row = knn + m * k;
    int lim = min(ei, row_len(row, k));
    for (int t = 0; t < lim; t++) {
        int32_t o = row[t];
        if (o < n) atomicAdd((unsigned long long *)&cnt[o], 1ull);
    }
}

// reverse keys of G_t into each node's segment, and every node's first source
template <typename LenT>
__global__ void sac_scatter_kernel(const int32_t *knn, const LenT *kd, int64_t n, int k, int ei,
                                   const int64_t *rev_off, int32_t *cursor, uint64_t *keys,
                                   int32_t *first_src) {
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    const int32_t *row = knn + m * k;
    int lim = min(ei, row_len(row, k));
    int32_t best = -1;
    int64_t bestc = 0;
    for (int t = 0; t < lim; t++) {
        int32_t o = row[t];
        if (o >= n) continue;
        int slot = atomicAdd(&cursor[o], 1);
        keys[rev_off[o] + slot] = make_key(len_ord(kd[m * k + t]), (uint32_t)m);
        int64_t c = rev_off[o + 1] - rev_off[o];
        if (best < 0 || c < bestc || (c == bestc && o < best)) {
            best = o;
            bestc = c;
        }
    }
    first_src[m] = best;
}

// One wave per node o over its sorted N(G_t, o) (rv_nb/rv_len at rev_off):
// counts the kept edges (WRITE false) or writes their keys at out_off[o].
template <typename LenT, bool WRITE>
__global__ void __launch_bounds__(256) sac_select_kernel(
    const int64_t *rev_off, const int32_t *rv_nb, const LenT *rv_len, const int32_t *first_src,
    const int32_t *knn, const LenT *kd, int64_t n, int k, int eo, int64_t *out_cnt,
    const int64_t *out_off, uint64_t *keys) {
    const int64_t o = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const int lane = lane_id();
    if (o >= n) return;
    const int64_t b = rev_off[o];
    const int m = (int)(rev_off[o + 1] - b);
    const int head = min(m, eo);
    const int64_t w = WRITE ? out_off[o] : 0;
    if (WRITE)
        for (int p = lane; p < head; p += WAVE)
            keys[w + p] = make_key(len_ord(rv_len[b + p]), (uint32_t)rv_nb[b + p]);
    int c = head;
    for (int p0 = head; p0 < m; p0 += WAVE) {
        const int p = p0 + lane;
        const bool keep = p < m && first_src[rv_nb[b + p]] == (int32_t)o;
        const uint64_t bal = ballot(keep);
        if (WRITE && keep)
            keys[w + c + mbcnt(bal)] = make_key(len_ord(rv_len[b + p]), (uint32_t)rv_nb[b + p]);
        c += __popcll(bal);
    }
    if (m < eo) {
        const int32_t *row = knn + o * k;
        const LenT *rd = kd + o * k;
        for (int t0 = 0; t0 < k && c < eo; t0 += WAVE) {
            const int t = t0 + lane;
            const int32_t id = t < k ? row[t] : -1;
            bool add = id >= 0;
            for (int p = 0; add && p < m; p++) add = rv_nb[b + p] != id;
            const uint64_t bal = ballot(add);
            const int r = c + mbcnt(bal);
            if (WRITE && add && r < eo) keys[w + r] = make_key(len_ord(rd[t]), (uint32_t)id);
            c = min(eo, c + __popcll(bal));
        }
    }
    if (!WRITE && lane == 0) out_cnt[o] = c;
}

// --------------------------------------------------------- Algorithms 4/5 --
// Round j of Algorithm 4 visits every node with more than j edges in ascending
// id; node v's j-th edge v -> nd (length L) is removed when HasPath finds
// v -> c and c -> nd in G_p with len(c, nd) < L.  At v's turn G_p holds the
// edges decided before (j, v) in lexicographic order, so with (v, i) the i-th
// edge of v's list, to c, and (c, jc) an edge of c's list to nd:
//   (v, j) is removed  iff  for some i < j and some (jc, c) < (j, v) with
//   len(c, jc) < L both (v, i) and (c, jc) are kept.
// Each decision depends on edges that precede it, so the decisions are the
// unique fixpoint of that rule, whatever order they are found in.  Every edge
// has a status (undecided, kept, removed) and a pass visits each node that
// still has undecided edges: a pair of kept edges removes (v, j), no pair
// without a removed member keeps it, anything else waits for the next pass.
// Statuses only ever become decided and a stale read (another node's write of
// the same pass not seen) reads "undecided", so the passes need no order
// among nodes.  The first undecided edge in (j, v) order is decided by every
// pass; in practice about ten passes decide all of them (200,003 x 100 cosine
// rows: 13.5M edges, longest list 2,734).
//
// A work item is up to CAP consecutive targets of one node's list: its
// undecided targets go into a hash table in LDS, and the lists of the node's
// not yet removed neighbours stream past it, coalesced, in pieces of 64 entries
// of which four are in flight.  Lists of at most 128 are one item of one wave, in rank order, so an
// edge kept by this very pass already serves as a witness; longer lists are
// cut into items of 512 targets, each taken by four waves in no order, which
// count only edges decided before.  Three quarters of a wave's time it waits for
// list pieces, scattered runs of some 270 bytes: 20 GB over all passes, at
// 2 TB/s.  Those 13.5M edges take 10.4 ms (11.7 with one list in flight; with a
// table whose buckets of four ids are one 16-byte LDS read 13.8; with one block
// size per class of list length, in three launches a pass, 15.2).  The earlier form ran one round per rank (as many as the
// longest list, each with a same-round settling pass and a host
// synchronisation) with a binary search per kept neighbour: 458 ms.

constexpr int8_t ST_UNDECIDED = 0, ST_KEPT = 1, ST_REMOVED = 2;
constexpr int64_t PA_MAX_DEGREE = (1 << 20) - 1;   // longer lists are refused
constexpr int PA_SMALL = 128;          // longest list that one wave takes
constexpr int PA_CHUNK = 512;          // targets per item of a longer list
constexpr int PA_AHEAD = 4;            // pieces of 64 list entries in flight per wave
constexpr uint32_t PA_EMPTY = 0xFFFFFFFFu;   // no node id (ids are below 2^31)

// The hash table has four slots per target, so that probe runs stay short; a
// repeated id takes several slots, and only then (dup) a lookup goes on past
// its first match.
template <typename LenT, int CAP, typename RankT>
struct PaTable {
    static constexpr int HSZ = 4 * CAP;
    uint32_t hid[HSZ];
    RankT hrank[HSZ];
    LenT len[CAP];
    uint8_t st[CAP];       // status before this pass
    uint8_t rem[CAP];      // a witness pair is kept
    uint8_t pend[CAP];     // a witness pair is not yet decided
    int32_t last;          // last undecided rank within the item
    int32_t dup;
    int32_t left, kept;    // targets still undecided, targets kept by this pass
    static __device__ uint32_t slot(uint32_t id) { return (id * 2654435761u) >> (32 - __builtin_ctz(HSZ)); }
    static __device__ uint32_t next(uint32_t h) { return (h + 1) & (HSZ - 1); }
};

template <typename T>
__device__ __forceinline__ T ld_relaxed(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <typename LenT>
struct PaGraph {
    const int64_t *off;
    const int32_t *nbrs;
    const LenT *lens;
    int64_t n;
    int8_t *st;            // status per edge
    int64_t *kept;         // kept edges per node
};

// One item: targets [t0, t0 + m) of node v, by WAVES waves (this one is w).
template <typename LenT, int CAP, typename RankT, int WAVES>
__device__ void pa_item(const PaGraph<LenT> &g, PaTable<LenT, CAP, RankT> &T, int32_t v, int t0,
                        int w, int32_t *left_at) {
    typedef PaTable<LenT, CAP, RankT> Table;
    constexpr int NT = WAVES * WAVE;
    const int lane = lane_id();
    const int tid = w * WAVE + lane;
    auto sync = [&]() {
        if constexpr (WAVES == 1) wave_sync();
        else __syncthreads();
    };
    const int64_t b = g.off[v];
    const int m = (int)min<int64_t>(CAP, g.off[v + 1] - b - t0);
    for (int i = tid; i < Table::HSZ; i += NT) T.hid[i] = PA_EMPTY;
    if (tid == 0) T.last = -1, T.dup = 0, T.left = 0, T.kept = 0;
    sync();
    int my_last = -1;
    for (int i = tid; i < m; i += NT) {
        const int8_t s = ld_relaxed(&g.st[b + t0 + i]);
        T.st[i] = (uint8_t)s;
        T.rem[i] = 0;
        T.pend[i] = 0;
        if (s == ST_UNDECIDED) {
            const uint32_t c = (uint32_t)g.nbrs[b + t0 + i];
            T.len[i] = g.lens[b + t0 + i];
            my_last = i;
            uint32_t h = Table::slot(c), was;
            while ((was = atomicCAS(&T.hid[h], PA_EMPTY, c)) != PA_EMPTY) {
                if (was == c) T.dup = 1;
                h = Table::next(h);
            }
            T.hrank[h] = (RankT)i;
        }
    }
    if (my_last >= 0) atomicMax(&T.last, my_last);
    sync();
    const int last = uni(T.last);
    const bool dup = uni(T.dup) != 0;
    const int lim = last < 0 ? 0 : t0 + last + 1;   // (c, jc) matters only for jc < lim
    // ranks below the last undecided target, 64 at a time: their neighbours'
    // lists are found by the lanes together, then taken one after another
    for (int ib = w * WAVE; ib < lim - 1; ib += NT) {
        const int il = ib + lane;
        int sl = ST_REMOVED;
        int32_t cl = -1;
        int64_t cbl = 0;
        int32_t cnl = 0;
        if (il < lim - 1) {
            sl = ld_relaxed(&g.st[b + il]);
            cl = g.nbrs[b + il];
            if (sl != ST_REMOVED && (uint32_t)cl < (uint64_t)g.n) {
                cbl = g.off[cl];
                cnl = (int32_t)min<int64_t>(g.off[cl + 1] - cbl, lim);
            }
        }
        // A unit is 64 entries of one list.  PA_AHEAD of them are in flight; the
        // loads are unconditional (lanes past the end read the last entry, past
        // the last unit the item's own list), so that the wait for one unit
        // leaves the later ones in flight.
        uint64_t todo = ballot(cnl > 0), ask = todo;
        int todo_j = 0, ask_j = 0;   // first entry of the unit to take, to request
        if (!todo) continue;
        int32_t x[PA_AHEAD];
        LenT lx[PA_AHEAD];
        uint32_t sx[PA_AHEAD];   // the word of the status (extending a byte would wait for it)
        auto request = [&](int d) __attribute__((always_inline)) {
            const int src = (int)__builtin_ctzll(ask | 1ull << 63);
            const int cn = __builtin_amdgcn_readlane(cnl, src);
            const int cnt = ask ? min(cn - ask_j, WAVE) : 1;
            const int64_t at = (ask ? readlane64(cbl, src) + ask_j : b) + min(lane, cnt - 1);
            x[d] = g.nbrs[at];
            lx[d] = g.lens[at];
            sx[d] = ld_relaxed(reinterpret_cast<const uint32_t *>(g.st) + (at >> 2));
            const bool more = ask && ask_j + WAVE < cn;
            ask = more ? ask : ask & (ask - 1);
            ask_j = more ? ask_j + WAVE : 0;
        };
#pragma unroll
        for (int d = 0; d < PA_AHEAD; d++) request(d);
        while (todo) {
#pragma unroll
            for (int d = 0; d < PA_AHEAD; d++) {
                if (!todo) break;
                const int src = (int)__builtin_ctzll(todo);
                const int i = ib + src;
                int si = __builtin_amdgcn_readlane(sl, src);
                const int32_t c = __builtin_amdgcn_readlane(cl, src);
                const int cn = __builtin_amdgcn_readlane(cnl, src);
                const int jc = todo_j + lane;
                bool look = jc < cn;
                if (si == ST_UNDECIDED && i >= t0) {
                    const int rem = T.rem[i - t0], pend = T.pend[i - t0];
                    look = look && !rem;
                    // one wave, in rank order: all that could hold it back has run
                    if (WAVES == 1 && !uni(pend)) si = ST_KEPT;
                }
                const int sy = (int)(sx[d] >> (((__builtin_amdgcn_readlane((int)cbl, src) + lane) & 3) * 8)) & 0xff;
                if (look && sy != ST_REMOVED) {
                    const uint32_t y = (uint32_t)x[d];
                    uint32_t h = Table::slot(y);
                    for (uint32_t id; (id = T.hid[h]) != PA_EMPTY; h = Table::next(h)) {
                        if (id != y) continue;
                        const int k = T.hrank[h];
                        const int j = t0 + k;
                        if (j > i && (jc < j || (jc == j && c < v)) && lx[d] < T.len[k]) {
                            if (si == ST_KEPT && sy == ST_KEPT) T.rem[k] = 1;
                            else T.pend[k] = 1;
                        }
                        if (!dup) break;
                    }
                }
                const bool more = todo_j + WAVE < cn;
                todo = more ? todo : todo & (todo - 1);
                todo_j = more ? todo_j + WAVE : 0;
                request(d);
                if constexpr (WAVES == 1) wave_sync();   // this unit's flags before the next status
            }
        }
    }
    sync();
    int nl = 0, nk = 0;
    for (int i = tid; i < m; i += NT) {
        if (T.st[i] != ST_UNDECIDED) continue;
        const int8_t s = T.rem[i] ? ST_REMOVED : T.pend[i] ? ST_UNDECIDED : ST_KEPT;
        if (s != ST_UNDECIDED)
            __hip_atomic_store(&g.st[b + t0 + i], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        nl += s == ST_UNDECIDED;
        nk += s == ST_KEPT;
    }
    if (nl) atomicAdd(&T.left, nl);
    if (nk) atomicAdd(&T.kept, nk);
    sync();
    if (tid == 0) {
        *left_at = T.left;
        if (T.kept) atomicAdd((unsigned long long *)&g.kept[v], (unsigned long long)T.kept);
    }
}

// One pass: the first n_big blocks take one item (node << 32 | chunk) of a
// long list each (they run longest), the others four short lists.
template <typename LenT>
__global__ void __launch_bounds__(256) pa_pass_kernel(PaGraph<LenT> g, const int64_t *big,
                                                      int64_t n_big, const int32_t *small,
                                                      int64_t n_small, int32_t *left_big,
                                                      int32_t *left_small) {
    typedef PaTable<LenT, PA_SMALL, uint8_t> SmallT;
    typedef PaTable<LenT, PA_CHUNK, uint16_t> BigT;
    __shared__ union {
        char small[4 * sizeof(SmallT)];
        char big[sizeof(BigT)];
    } lds;
    static_assert(alignof(SmallT) == 4 && alignof(BigT) == 4 && sizeof(SmallT) % 4 == 0, "LDS layout");
    const int wv = uni(threadIdx.x / WAVE);
    if (blockIdx.x < n_big) {
        const int64_t it = (int64_t)uni64((uint64_t)big[blockIdx.x]);
        pa_item<LenT, PA_CHUNK, uint16_t, 4>(g, *reinterpret_cast<BigT *>(lds.big),
                                             (int32_t)(it >> 32), (int)(uint32_t)it * PA_CHUNK, wv,
                                             left_big + blockIdx.x);
        return;
    }
    // consecutive nodes share neighbours: give each XCD (blocks go to the 8 XCDs
    // in turn) one run of the list
    const int64_t nblk = gridDim.x - n_big, per = nblk / 8, rest = nblk - per * 8;
    const int64_t xcd = (blockIdx.x - n_big) % 8, at = (blockIdx.x - n_big) / 8;
    const int64_t gi = (xcd * per + min(xcd, rest) + at) * 4 + wv;
    if (gi >= n_small) return;
    pa_item<LenT, PA_SMALL, uint8_t, 1>(g, reinterpret_cast<SmallT *>(lds.small)[wv],
                                        uni(small[gi]), 0, 0, left_small + gi);
}

// The first pass's items, all lists: counters[0] short lists, counters[1]
// items of longer ones, counters[3] lists that are too long.
__global__ void __launch_bounds__(256) pa_items_kernel(const int64_t *off, int64_t n,
                                                       int32_t *small, int64_t *big,
                                                       unsigned long long *counters) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t deg = v < n ? off[v + 1] - off[v] : 0;
    const bool sm = deg > 0 && deg <= PA_SMALL;
    const uint64_t m = ballot(sm);
    if (m) {
        const int lead = (int)__builtin_ctzll(m);
        uint64_t at = 0;
        if (lane_id() == lead) at = atomicAdd(&counters[0], (unsigned long long)__popcll(m));
        at = shfl64(at, lead);
        if (sm) small[at + mbcnt(m)] = (int32_t)v;
    }
    if (deg > PA_SMALL) {
        if (deg >= PA_MAX_DEGREE) {
            atomicAdd(&counters[3], 1ull);
            return;
        }
        const int nc = (int)((deg + PA_CHUNK - 1) / PA_CHUNK);
        const unsigned long long at = atomicAdd(&counters[1], (unsigned long long)nc);
        for (int c = 0; c < nc; c++) big[at + c] = v << 32 | c;
    }
}

// The next pass's items: those with targets left; counters[2] the targets.
// The first `sb` blocks take the short lists.
__global__ void __launch_bounds__(256) pa_next_kernel(const int32_t *small, int64_t n_small,
                                                      const int32_t *left_small, int64_t sb,
                                                      const int64_t *big, int64_t n_big,
                                                      const int32_t *left_big, int32_t *next_small,
                                                      int64_t *next_big,
                                                      unsigned long long *counters) {
    const bool is_big = blockIdx.x >= sb;
    const int64_t i = (int64_t)(blockIdx.x - (is_big ? sb : 0)) * blockDim.x + threadIdx.x;
    const int64_t cnt = is_big ? n_big : n_small;
    int left = i < cnt ? (is_big ? left_big : left_small)[i] : 0;
    const uint64_t m = ballot(left > 0);
    if (!m) return;
    const int lead = (int)__builtin_ctzll(m);
    uint64_t at = 0;
    if (lane_id() == lead) at = atomicAdd(&counters[is_big], (unsigned long long)__popcll(m));
    at = shfl64(at, lead);
    if (left > 0) {
        if (is_big) next_big[at + mbcnt(m)] = big[i];
        else next_small[at + mbcnt(m)] = small[i];
    }
    for (int s = 32; s >= 1; s >>= 1) left += __shfl_xor(left, s);
    if (lane_id() == lead) atomicAdd(&counters[2], (unsigned long long)left);
}

// kept edges of every node, in list order (one wave per node)
template <typename LenT>
__global__ void __launch_bounds__(256) pa_compact_kernel(const int64_t *off, const int64_t *out_off,
                                                         int64_t n, const int32_t *nbrs,
                                                         const LenT *lens, const int8_t *st,
                                                         int32_t *out_nb, LenT *out_len) {
    const int64_t v = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
    const int lane = lane_id();
    if (v >= n) return;
    const int64_t b = off[v], e = off[v + 1];
    int64_t o = out_off[v];
    for (int64_t t = b; t < e; t += WAVE) {
        const bool keep = t + lane < e && st[t + lane] == ST_KEPT;
        const uint64_t m = ballot(keep);
        if (keep) {
            out_nb[o + mbcnt(m)] = nbrs[t + lane];
            out_len[o + mbcnt(m)] = lens[t + lane];
        }
        o += __popcll(m);
    }
}

__global__ void cnt_to_i64_kernel(const int32_t *c, int64_t n, int64_t *o) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) o[v] = c[v];
    if (v == n) o[n] = 0;
}

inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

size_t scan_temp_bytes(int64_t n) {
    size_t bytes = 0;
    (void)hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, (int64_t *)nullptr, (int64_t *)nullptr,
                                     (int)n);
    return bytes;
}

// ------------------------------------------------------ graph statistics --
// Degree shape and incoming-edge lengths of a graph (Table 4).

__global__ void gs_degree_kernel(const int64_t *off, const int32_t *nbrs, int64_t n,
                                 int32_t *outdeg, int32_t *indeg) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    outdeg[v] = (int32_t)(off[v + 1] - off[v]);
    for (int64_t e = off[v]; e < off[v + 1]; e++) {
        const int32_t t = nbrs[e];
        if (t >= 0 && t < n) atomicAdd(&indeg[t], 1);   // ids outside the graph count nowhere
    }
}

// every edge's length key into its target's segment of the transposed graph
template <typename LenT>
__global__ void gs_transpose_kernel(const int64_t *off, const int32_t *nbrs, const LenT *lens,
                                    int64_t n, const int64_t *toff, int32_t *cursor,
                                    uint32_t *tkeys) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    for (int64_t e = off[v]; e < off[v + 1]; e++) {
        const int32_t t = nbrs[e];
        if (t < 0 || t >= n) continue;
        const int slot = atomicAdd(&cursor[t], 1);
        tkeys[toff[t] + slot] = len_ord(lens[e]);
    }
}

// per node: the sum of its `keep` shortest incoming lengths, as distances
template <typename LenT, bool SQRT>
__global__ void gs_keep_kernel(const int64_t *toff, const uint32_t *sorted, int64_t n, int keep,
                               double *psum, double *pcnt) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    int64_t b = toff[v];
    int c = (int)min<int64_t>(keep, toff[v + 1] - b);
    double s = 0.0;
    for (int i = 0; i < c; i++) {
        uint32_t key = sorted[b + i];
        double x;
        if constexpr (std::is_integral<LenT>::value) x = (double)key;
        else x = (double)unord_f32(key);
        s += SQRT ? sqrt(x) : x;
    }
    psum[v] = s;
    pcnt[v] = (double)c;
}

// one block: out[slot] = sum of a[0 .. cnt) in double, in a fixed order
template <typename T>
__global__ void __launch_bounds__(1024) gs_sum_kernel(const T *a, int64_t cnt, double *out,
                                                      int slot) {
    __shared__ double part[1024];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < cnt; i += blockDim.x) s += (double)a[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[slot] = part[0];
}

__global__ void gs_final_kernel(const double *sums, double t, double *res) {
    res[0] = t > 0 ? sums[0] / t : 0.0;
    res[1] = t > 0 ? sums[1] / t : 0.0;
    res[2] = sums[3] > 0 ? sums[2] / sums[3] : 0.0;
}

// ------------------------------------------------------- edge insertion --
// Graph plus new edges (src, dst, length): per-node counts, offsets, keys of
// the old and new edges in each node's segment, then the (length, id) sort.

__global__ void ae_count_kernel(const int64_t *off, int64_t n, const int32_t *src,
                                const int32_t *dst, int64_t m, int64_t *cnt) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) atomicAdd((unsigned long long *)&cnt[i], (unsigned long long)(off[i + 1] - off[i]));
    if (i < m && src[i] >= 0 && src[i] < n && dst[i] >= 0 && dst[i] < n)
        atomicAdd((unsigned long long *)&cnt[src[i]], 1ull);
}

template <typename LenT>
__global__ void ae_scatter_kernel(const int64_t *off, const int32_t *nbrs, const LenT *lens,
                                  int64_t n, const int32_t *src, const int32_t *dst,
                                  const LenT *len, int64_t m, const int64_t *out_off,
                                  int32_t *cursor, uint64_t *keys) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const int64_t b = off[i], e = off[i + 1];
        const int64_t w = out_off[i];
        for (int64_t t = b; t < e; t++) keys[w + (t - b)] = make_key(len_ord(lens[t]), (uint32_t)nbrs[t]);
        cursor[i] = (int32_t)(e - b);
    }
}

template <typename LenT>
__global__ void ae_new_kernel(int64_t n, const int32_t *src, const int32_t *dst, const LenT *len,
                              int64_t m, const int64_t *out_off, int32_t *cursor, uint64_t *keys) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    const int32_t s = src[i], d = dst[i];
    if (s < 0 || s >= n || d < 0 || d >= n) return;
    const int slot = atomicAdd(&cursor[s], 1);
    keys[out_off[s] + slot] = make_key(len_ord(len[i]), (uint32_t)d);
}

}  // namespace

// ------------------------------------------------------------- host side --

// Sorts every list (see seg_sort_kernel); queue: n ints; n_queue: its length, zero.
template <typename LenT>
static void seg_sort(const int64_t *seg, const int64_t *off, int64_t n, const uint64_t *keys,
                     int32_t *nbrs, LenT *lens, int32_t *queue, int32_t *n_queue, hipStream_t st) {
    if (n == 0) return;
    if (n <= SEG_BLOCKS) {   // one launch for two: some 5 us of a call of 110 on 1000 nodes
        hipLaunchKernelGGL((seg_sort_long_kernel<LenT>), dim3((unsigned)n), dim3(512), 0, st, seg, off, keys,
                           nbrs, lens, nullptr, nullptr, (int)n);
        return;
    }
    hipLaunchKernelGGL((seg_sort_kernel<LenT>), dim3(blocks_for(n, 4)), dim3(256), 0, st, seg, off,
                       n, keys, nbrs, lens, queue, n_queue);
    hipLaunchKernelGGL((seg_sort_long_kernel<LenT>),
                       dim3(SEG_BLOCKS), dim3(512), 0, st, seg, off, keys, nbrs, lens, queue,
                       n_queue, 0);
}

// zeroes of consecutive regions of a workspace, first to end: one launch
static hipError_t clear_range(void *first, void *end, hipStream_t st) {
    return hipMemsetAsync(first, 0, (size_t)(static_cast<char *>(end) - static_cast<char *>(first)), st);
}

// The place behind the counts of n lists, zero for the scan, is the counter of the
// lists' sort afterwards.
static int32_t *zero_after_scan(int64_t *last) { return reinterpret_cast<int32_t *>(last); }

size_t adjust_degree_ws(int64_t n, int32_t k, int32_t e_o, int32_t e_i) {
    const int64_t eo = std::min(e_o, k), ei = std::min(e_i, k);
    Carver c(nullptr);
    c.take<int32_t>(n);                // reverse candidates per node
    c.take<int64_t>(n + 1);            // segment sizes, then edges per node
    c.take<int32_t>(n);                // forward edges per node
    c.take<int32_t>(n * ei);           // place of each reverse candidate
    c.take<int64_t>(n + 1);            // segment offsets
    c.take<uint64_t>(n * (eo + ei));   // keys
    c.take<int32_t>(n);                // long lists
    c.take<char>(scan_temp_bytes(n + 1));
    return c.size() + 256;
}

template <typename LenT>
static onng_status adjust_degree_impl(const int32_t *knn, const LenT *kd, int64_t n, int32_t k,
                                      int32_t e_o, int32_t e_i, int64_t *offsets, int32_t *nbrs,
                                      LenT *lens, int64_t nnz_cap, int64_t *nnz_out, void *ws,
                                      hipStream_t st) {
    const int eo = std::min(e_o, k), ei = std::min(e_i, k);
    Carver c(ws);
    int32_t *rcnt = c.take<int32_t>(n);
    int64_t *cnt = c.take<int64_t>(n + 1);
    int32_t *fcnt = c.take<int32_t>(n);
    int32_t *slot = c.take<int32_t>(n * (int64_t)ei);
    int64_t *seg = c.take<int64_t>(n + 1);
    uint64_t *keys = c.take<uint64_t>(n * (int64_t)(eo + ei));
    int32_t *queue = c.take<int32_t>(n);
    size_t tb = scan_temp_bytes(n + 1);
    void *tmp = c.take<char>(tb);
    const unsigned wb = blocks_for(n, 4);
    const bool short_rows =
        n == 0 || (std::max(eo, ei) <= SA_SHORT && n * std::max(eo, 1) * std::max(ei, 1) < 100000);
    ONNG_HIP(clear_range(rcnt, short_rows ? static_cast<void *>(cnt + n + 1) : rcnt + n, st));
    if (short_rows) {
        const dim3 grid(blocks_for(n, 256)), block(256);
        if (n > 0) hipLaunchKernelGGL(sa_short_count_kernel, grid, block, 0, st, knn, n, k, eo, ei, cnt);
        ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt, offsets, (int)(n + 1), st));
        if (n > 0)
            hipLaunchKernelGGL((sa_short_scatter_kernel<LenT>), grid, block, 0, st, knn, kd, n, k, eo, ei, offsets,
                               rcnt, keys);
    } else {
        hipLaunchKernelGGL(sa_count_kernel, dim3(blocks_for(n, SA_ROWS)), dim3(SA_WAVES * WAVE), 0, st, knn, n, k, eo,
                           ei, rcnt, slot, fcnt);
        hipLaunchKernelGGL(sa_sizes_kernel, dim3(blocks_for(n + 1, 256)), dim3(256), 0, st, rcnt, fcnt, n, cnt);
        ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt, seg, (int)(n + 1), st));
        hipLaunchKernelGGL((sa_scatter_kernel<LenT>), dim3(wb), dim3(256), 0, st, knn, kd, n, k, ei, seg, slot, keys);
        hipLaunchKernelGGL((sa_merge_kernel<LenT>), dim3(wb), dim3(256), 0, st, knn, kd, n, k, rcnt, fcnt, seg, keys,
                           cnt);
        ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt, offsets, (int)(n + 1), st));
    }
    ONNG_HIP(hipMemcpyAsync(nnz_out, offsets + n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    ONNG_HIP(hipStreamSynchronize(st));
    if (*nnz_out > nnz_cap) {
        set_error("onng_adjust_degree: nnz_capacity too small");
        return ONNG_ERR_CAPACITY;
    }
    seg_sort<LenT>(short_rows ? offsets : seg, offsets, n, keys, nbrs, lens, queue, zero_after_scan(cnt + n), st);
    ONNG_HIP(hipGetLastError());
    ONNG_HIP(hipStreamSynchronize(st));
    return ONNG_OK;
}

onng_status adjust_degree_launch(const int32_t *knn, const void *kd, int64_t n, int32_t k,
                                 bool int_len, int32_t e_o, int32_t e_i, int64_t *offsets,
                                 int32_t *nbrs, void *lens, int64_t nnz_cap, int64_t *nnz_out,
                                 void *ws, hipStream_t st) {
    if (int_len)
        return adjust_degree_impl<int32_t>(knn, static_cast<const int32_t *>(kd), n, k, e_o, e_i,
                                           offsets, nbrs, static_cast<int32_t *>(lens), nnz_cap,
                                           nnz_out, ws, st);
    return adjust_degree_impl<float>(knn, static_cast<const float *>(kd), n, k, e_o, e_i, offsets,
                                     nbrs, static_cast<float *>(lens), nnz_cap, nnz_out, ws, st);
}

size_t adjust_degree_constrained_ws(int64_t n, int32_t k, int32_t e_o, int32_t e_i) {
    const int64_t nrev = n * (int64_t)std::min(e_i, k);
    const int64_t cap = nrev + n * (int64_t)std::min(e_o, k);
    Carver c(nullptr);
    c.take<int64_t>(n + 1);            // |N(G_t, o)|
    c.take<int64_t>(n + 1);            // kept counts
    c.take<int32_t>(n);                // cursors
    c.take<int64_t>(n + 1);            // G_t offsets
    c.take<int32_t>(n);                // first source per node
    c.take<uint64_t>(nrev);            // G_t keys
    c.take<int32_t>(nrev);             // G_t ids, sorted per node
    c.take<int32_t>(nrev);             // G_t lengths (4 bytes)
    c.take<uint64_t>(cap);             // kept keys
    c.take<int32_t>(n);                // long lists
    c.take<char>(scan_temp_bytes(n + 1));
    return c.size() + 256;
}

template <typename LenT>
static onng_status adjust_degree_constrained_impl(const int32_t *knn, const LenT *kd, int64_t n,
                                                  int32_t k, int32_t e_o, int32_t e_i,
                                                  int64_t *offsets, int32_t *nbrs, LenT *lens,
                                                  int64_t nnz_cap, int64_t *nnz_out, void *ws,
                                                  hipStream_t st) {
    const int ei = std::min(e_i, k);
    const int eo = e_o;
    const int64_t nrev = n * (int64_t)ei;
    const int64_t cap = nrev + n * (int64_t)std::min(e_o, k);
    Carver c(ws);
    int64_t *cnt = c.take<int64_t>(n + 1);
    int64_t *ocnt = c.take<int64_t>(n + 1);
    int32_t *cursor = c.take<int32_t>(n);
    int64_t *rev_off = c.take<int64_t>(n + 1);
    int32_t *first_src = c.take<int32_t>(n);
    uint64_t *rkeys = c.take<uint64_t>(nrev);
    int32_t *rv_nb = c.take<int32_t>(nrev);
    LenT *rv_len = reinterpret_cast<LenT *>(c.take<int32_t>(nrev));
    uint64_t *okeys = c.take<uint64_t>(cap);
    int32_t *queue = c.take<int32_t>(n);
    size_t tb = scan_temp_bytes(n + 1);
    void *tmp = c.take<char>(tb);
    ONNG_HIP(clear_range(cnt, cursor + n, st));
    if (n > 0) {
        hipLaunchKernelGGL(sac_rcount_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, knn, n,
                           k, ei, cnt);
        ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt, rev_off, (int)(n + 1), st));
        hipLaunchKernelGGL((sac_scatter_kernel<LenT>), dim3(blocks_for(n, 256)), dim3(256), 0, st,
                           knn, kd, n, k, ei, rev_off, cursor, rkeys, first_src);
        seg_sort<LenT>(rev_off, rev_off, n, rkeys, rv_nb, rv_len, queue, zero_after_scan(cnt + n), st);
        hipLaunchKernelGGL((sac_select_kernel<LenT, false>), dim3(blocks_for(n * WAVE, 256)),
                           dim3(256), 0, st, rev_off, rv_nb, rv_len, first_src, knn, kd, n, k, eo,
                           ocnt, nullptr, nullptr);
        ONNG_HIP(hipGetLastError());
    }
    ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, ocnt, offsets, (int)(n + 1), st));
    ONNG_HIP(hipMemcpyAsync(nnz_out, offsets + n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    ONNG_HIP(hipStreamSynchronize(st));
    if (*nnz_out > nnz_cap) {
        set_error("onng_adjust_degree_constrained: nnz_capacity too small");
        return ONNG_ERR_CAPACITY;
    }
    if (*nnz_out > cap) {
        set_error("onng_adjust_degree_constrained: more edges than the workspace bound");
        return ONNG_ERR_CAPACITY;
    }
    if (n > 0) {
        hipLaunchKernelGGL((sac_select_kernel<LenT, true>), dim3(blocks_for(n * WAVE, 256)),
                           dim3(256), 0, st, rev_off, rv_nb, rv_len, first_src, knn, kd, n, k, eo,
                           nullptr, offsets, okeys);
        seg_sort<LenT>(offsets, offsets, n, okeys, nbrs, lens, queue, zero_after_scan(ocnt + n), st);
    }
    ONNG_HIP(hipGetLastError());
    ONNG_HIP(hipStreamSynchronize(st));
    return ONNG_OK;
}

onng_status adjust_degree_constrained_launch(const int32_t *knn, const void *kd, int64_t n,
                                             int32_t k, bool int_len, int32_t e_o, int32_t e_i,
                                             int64_t *offsets, int32_t *nbrs, void *lens,
                                             int64_t nnz_cap, int64_t *nnz_out, void *ws,
                                             hipStream_t st) {
    if (int_len)
        return adjust_degree_constrained_impl<int32_t>(
            knn, static_cast<const int32_t *>(kd), n, k, e_o, e_i, offsets, nbrs,
            static_cast<int32_t *>(lens), nnz_cap, nnz_out, ws, st);
    return adjust_degree_constrained_impl<float>(knn, static_cast<const float *>(kd), n, k, e_o,
                                                 e_i, offsets, nbrs, static_cast<float *>(lens),
                                                 nnz_cap, nnz_out, ws, st);
}

static size_t gs_sort_temp_bytes(int64_t n, int64_t nnz) {
    size_t a = 0, b = 0, d = 0;
    (void)hipcub::DeviceRadixSort::SortKeys(nullptr, a, (const int32_t *)nullptr,
                                            (int32_t *)nullptr, (int)n);
    (void)hipcub::DeviceRadixSort::SortKeysDescending(nullptr, d, (const int32_t *)nullptr,
                                                      (int32_t *)nullptr, (int)n);
    a = std::max(a, d);
    (void)hipcub::DeviceSegmentedRadixSort::SortKeys(
        nullptr, b, (const uint32_t *)nullptr, (uint32_t *)nullptr, (int)nnz, (int)n,
        (const int64_t *)nullptr, (const int64_t *)nullptr);
    return std::max(std::max(a, b), scan_temp_bytes(n + 1));
}

size_t graph_stats_ws(int64_t n, int64_t nnz) {
    Carver c(nullptr);
    c.take<int32_t>(n);          // out-degrees
    c.take<int32_t>(n);          // in-degrees
    c.take<int32_t>(n);          // sorted degrees
    c.take<int32_t>(n);          // cursors
    c.take<int64_t>(n + 1);      // in-degrees as int64
    c.take<int64_t>(n + 1);      // transposed offsets
    c.take<uint32_t>(nnz);       // incoming length keys
    c.take<uint32_t>(nnz);       // the same, sorted per node
    c.take<double>(n);           // per-node sums
    c.take<double>(n);           // per-node counts
    c.take<double>(8);           // sums and results
    c.take<char>(gs_sort_temp_bytes(n, nnz));
    return c.size() + 256;
}

template <typename LenT>
static onng_status graph_stats_impl(const onng_graph *g, bool sqrt_len, double frac, int keep,
                                    double *out, void *ws, hipStream_t st) {
    const int64_t n = g->n, nnz = g->nnz;
    Carver c(ws);
    int32_t *outdeg = c.take<int32_t>(n);
    int32_t *indeg = c.take<int32_t>(n);
    int32_t *sdeg = c.take<int32_t>(n);
    int32_t *cursor = c.take<int32_t>(n);
    int64_t *in64 = c.take<int64_t>(n + 1);
    int64_t *toff = c.take<int64_t>(n + 1);
    uint32_t *tkeys = c.take<uint32_t>(nnz);
    uint32_t *tsorted = c.take<uint32_t>(nnz);
    double *psum = c.take<double>(n);
    double *pcnt = c.take<double>(n);
    double *sums = c.take<double>(8);
    size_t tb = gs_sort_temp_bytes(n, nnz);
    void *tmp = c.take<char>(tb);
    const int64_t t = n > 0 ? std::max<int64_t>(1, (int64_t)std::floor(frac * (double)n)) : 0;
    ONNG_HIP(hipMemsetAsync(indeg, 0, sizeof(int32_t) * n, st));
    ONNG_HIP(hipMemsetAsync(cursor, 0, sizeof(int32_t) * n, st));
    ONNG_HIP(hipMemsetAsync(sums, 0, sizeof(double) * 8, st));
    if (n > 0) {
        const unsigned nb = blocks_for(n, 256);
        hipLaunchKernelGGL(gs_degree_kernel, dim3(nb), dim3(256), 0, st, g->offsets, g->nbrs, n,
                           outdeg, indeg);
        size_t b = tb;
        ONNG_HIP(hipcub::DeviceRadixSort::SortKeysDescending(tmp, b, outdeg, sdeg, (int)n, 0, 32,
                                                             st));
        hipLaunchKernelGGL((gs_sum_kernel<int32_t>), dim3(1), dim3(1024), 0, st, sdeg, t, sums, 0);
        b = tb;
        ONNG_HIP(hipcub::DeviceRadixSort::SortKeys(tmp, b, indeg, sdeg, (int)n, 0, 32, st));
        hipLaunchKernelGGL((gs_sum_kernel<int32_t>), dim3(1), dim3(1024), 0, st, sdeg, t, sums, 1);
        hipLaunchKernelGGL(cnt_to_i64_kernel, dim3(blocks_for(n + 1, 256)), dim3(256), 0, st,
                           indeg, n, in64);
        b = tb;
        ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, b, in64, toff, (int)(n + 1), st));
        hipLaunchKernelGGL((gs_transpose_kernel<LenT>), dim3(nb), dim3(256), 0, st, g->offsets,
                           g->nbrs, static_cast<const LenT *>(g->lens), n, toff, cursor, tkeys);
        if (nnz > 0) {
            b = tb;
            ONNG_HIP(hipcub::DeviceSegmentedRadixSort::SortKeys(
                tmp, b, tkeys, tsorted, (int)nnz, (int)n, toff, toff + 1, 0, 32, st));
        }
        if (sqrt_len)
            hipLaunchKernelGGL((gs_keep_kernel<LenT, true>), dim3(nb), dim3(256), 0, st, toff,
                               tsorted, n, keep, psum, pcnt);
        else
            hipLaunchKernelGGL((gs_keep_kernel<LenT, false>), dim3(nb), dim3(256), 0, st, toff,
                               tsorted, n, keep, psum, pcnt);
        hipLaunchKernelGGL((gs_sum_kernel<double>), dim3(1), dim3(1024), 0, st, psum, n, sums, 2);
        hipLaunchKernelGGL((gs_sum_kernel<double>), dim3(1), dim3(1024), 0, st, pcnt, n, sums, 3);
    }
    hipLaunchKernelGGL(gs_final_kernel, dim3(1), dim3(1), 0, st, sums, (double)t, sums + 4);
    ONNG_HIP(hipGetLastError());
    ONNG_HIP(hipMemcpyAsync(out, sums + 4, 3 * sizeof(double), hipMemcpyDeviceToHost, st));
    ONNG_HIP(hipStreamSynchronize(st));
    return ONNG_OK;
}

onng_status graph_stats_launch(const onng_graph *g, bool int_len, bool sqrt_len, double frac,
                               int keep, double *out, void *ws, hipStream_t st) {
    if (int_len) return graph_stats_impl<int32_t>(g, sqrt_len, frac, keep, out, ws, st);
    return graph_stats_impl<float>(g, sqrt_len, frac, keep, out, ws, st);
}

// ---------------------------------------------- first k edges of a graph --

namespace {

// Row v of the table: the first min(k, deg(v)) edges of v's list (sorted by
// (length, id)), then padding (-1, INT32_MAX or +inf).  One lane per entry.
template <typename LT>
__global__ void graph_head_kernel(const int64_t *off, const int32_t *nb, const LT *len, int64_t n,
                                  int32_t k, LT pad, int32_t *ids, LT *dists) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * (int64_t)k) return;
    const int64_t v = t / k;
    const int32_t j = (int32_t)(t - v * k);
    const int64_t e = off[v] + j;
    const bool has = e < off[v + 1];
    ids[t] = has ? nb[e] : -1;
    dists[t] = has ? len[e] : pad;
}

}  // namespace

onng_status graph_head_launch(const onng_graph *g, bool int_len, int32_t k, int32_t *ids,
                              void *dists, hipStream_t st) {
    const int64_t total = g->n * (int64_t)k;
    if (total == 0) return ONNG_OK;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (int_len)
        hipLaunchKernelGGL(graph_head_kernel<int32_t>, dim3(blocks), dim3(256), 0, st, g->offsets,
                           g->nbrs, static_cast<const int32_t *>(g->lens), g->n, k, INT32_MAX, ids,
                           static_cast<int32_t *>(dists));
    else
        hipLaunchKernelGGL(graph_head_kernel<float>, dim3(blocks), dim3(256), 0, st, g->offsets,
                           g->nbrs, static_cast<const float *>(g->lens), g->n, k,
                           __builtin_huge_valf(), ids, static_cast<float *>(dists));
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

size_t add_edges_ws(int64_t n, int64_t nnz, int64_t m) {
    Carver c(nullptr);
    c.take<int64_t>(n + 1);
    c.take<int32_t>(n);
    c.take<uint64_t>(nnz + m);
    c.take<int32_t>(n);
    c.take<char>(scan_temp_bytes(n + 1));
    return c.size() + 256;
}

template <typename LenT>
static onng_status add_edges_impl(const onng_graph *g, const int32_t *src, const int32_t *dst,
                                  const LenT *len, int64_t m, int64_t *out_off, int32_t *out_nb,
                                  LenT *out_len, int64_t nnz_cap, int64_t *nnz_out, void *ws,
                                  hipStream_t st) {
    const int64_t n = g->n, nnz = g->nnz;
    Carver c(ws);
    int64_t *cnt = c.take<int64_t>(n + 1);
    int32_t *cursor = c.take<int32_t>(n);
    uint64_t *keys = c.take<uint64_t>(nnz + m);
    int32_t *queue = c.take<int32_t>(n);
    size_t tb = scan_temp_bytes(n + 1);
    void *tmp = c.take<char>(tb);
    ONNG_HIP(clear_range(cnt, cursor + n, st));
    const int64_t big = std::max(n, m);
    if (big > 0)
        hipLaunchKernelGGL(ae_count_kernel, dim3(blocks_for(big, 256)), dim3(256), 0, st,
                           g->offsets, n, src, dst, m, cnt);
    ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt, out_off, (int)(n + 1), st));
    ONNG_HIP(hipMemcpyAsync(nnz_out, out_off + n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    ONNG_HIP(hipStreamSynchronize(st));
    if (*nnz_out > nnz_cap) {
        set_error("onng_graph_add_edges: nnz_capacity too small");
        return ONNG_ERR_CAPACITY;
    }
    if (n > 0) {
        hipLaunchKernelGGL((ae_scatter_kernel<LenT>), dim3(blocks_for(n, 256)), dim3(256), 0, st,
                           g->offsets, g->nbrs, static_cast<const LenT *>(g->lens), n, src, dst,
                           len, m, out_off, cursor, keys);
        if (m > 0)
            hipLaunchKernelGGL((ae_new_kernel<LenT>), dim3(blocks_for(m, 256)), dim3(256), 0, st,
                               n, src, dst, len, m, out_off, cursor, keys);
        seg_sort<LenT>(out_off, out_off, n, keys, out_nb, out_len, queue, zero_after_scan(cnt + n), st);
    }
    ONNG_HIP(hipGetLastError());
    ONNG_HIP(hipStreamSynchronize(st));
    return ONNG_OK;
}

onng_status add_edges_launch(const onng_graph *g, const int32_t *src, const int32_t *dst,
                             const void *len, int64_t m, bool int_len, int64_t *out_off,
                             int32_t *out_nb, void *out_len, int64_t nnz_cap, int64_t *nnz_out,
                             void *ws, hipStream_t st) {
    if (int_len)
        return add_edges_impl<int32_t>(g, src, dst, static_cast<const int32_t *>(len), m, out_off,
                                       out_nb, static_cast<int32_t *>(out_len), nnz_cap, nnz_out,
                                       ws, st);
    return add_edges_impl<float>(g, src, dst, static_cast<const float *>(len), m, out_off, out_nb,
                                 static_cast<float *>(out_len), nnz_cap, nnz_out, ws, st);
}

// items of lists longer than PA_SMALL: ceil(deg / PA_CHUNK) of each
static int64_t pa_big_cap(int64_t nnz) { return nnz / PA_SMALL + nnz / PA_CHUNK + 1; }

size_t adjust_path_ws(int64_t n, int64_t nnz) {
    const int64_t nb = pa_big_cap(nnz);
    Carver c(nullptr);
    c.take<int8_t>(nnz);                // status per edge
    c.take<int32_t>(n);                 // short lists, this and the next pass
    c.take<int32_t>(n);
    c.take<int64_t>(nb);                // items of long lists, likewise
    c.take<int64_t>(nb);
    c.take<int32_t>(n);                 // undecided targets per short list
    c.take<int32_t>(nb);                // ... per item of a long list
    c.take<unsigned long long>(4);      // counters
    c.take<int64_t>(n + 1);             // kept edges per node
    c.take<char>(scan_temp_bytes(n + 1));
    return c.size() + 256;
}

template <typename LenT>
static onng_status adjust_path_impl(const onng_graph *g, int64_t *out_off, int32_t *out_nb,
                                    LenT *out_len, int64_t *nnz_out, void *ws, hipStream_t st) {
    const int64_t n = g->n, nnz = g->nnz, nb = pa_big_cap(nnz);
    const LenT *lens = static_cast<const LenT *>(g->lens);
    Carver c(ws);
    int8_t *status = c.take<int8_t>(nnz);
    int32_t *small[2];
    int64_t *big[2];
    for (int32_t *&l : small) l = c.take<int32_t>(n);
    for (int64_t *&l : big) l = c.take<int64_t>(nb);
    int32_t *left_small = c.take<int32_t>(n);
    int32_t *left_big = c.take<int32_t>(nb);
    unsigned long long *counters = c.take<unsigned long long>(4);
    int64_t *kept = c.take<int64_t>(n + 1);
    size_t tb = scan_temp_bytes(n + 1);
    void *tmp = c.take<char>(tb);
    const PaGraph<LenT> pg{g->offsets, g->nbrs, lens, n, status, kept};
    ONNG_HIP(hipMemsetAsync(status, ST_UNDECIDED, (size_t)nnz, st));
    ONNG_HIP(hipMemsetAsync(kept, 0, sizeof(int64_t) * (n + 1), st));
    ONNG_HIP(hipMemsetAsync(counters, 0, sizeof(unsigned long long) * 4, st));
    unsigned long long h[4] = {0, 0, 0, 0};
    if (n > 0) {
        hipLaunchKernelGGL(pa_items_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, g->offsets,
                           n, small[0], big[0], counters);
        ONNG_HIP(hipMemcpyAsync(h, counters, sizeof(h), hipMemcpyDeviceToHost, st));
        ONNG_HIP(hipStreamSynchronize(st));
    }
    if (h[3]) {
        set_error("onng_adjust_path: a node has 2^20 - 1 or more edges");
        return ONNG_ERR_UNSUPPORTED;
    }
    unsigned long long before = (unsigned long long)nnz + 1;
    for (int side = 0; h[0] + h[1] > 0; side ^= 1) {
        const int64_t ns = (int64_t)h[0], nbig = (int64_t)h[1];
        ONNG_HIP(hipMemsetAsync(counters, 0, sizeof(unsigned long long) * 4, st));
        hipLaunchKernelGGL((pa_pass_kernel<LenT>), dim3((unsigned)nbig + blocks_for(ns, 4)),
                           dim3(256), 0, st, pg, big[side], nbig, small[side], ns, left_big,
                           left_small);
        const unsigned sb = blocks_for(ns, 256);
        hipLaunchKernelGGL(pa_next_kernel, dim3(sb + blocks_for(nbig, 256)), dim3(256), 0, st,
                           small[side], ns, left_small, (int64_t)sb, big[side], nbig, left_big,
                           small[side ^ 1], big[side ^ 1], counters);
        ONNG_HIP(hipGetLastError());
        ONNG_HIP(hipMemcpyAsync(h, counters, sizeof(h), hipMemcpyDeviceToHost, st));
        ONNG_HIP(hipStreamSynchronize(st));
        if (h[2] >= before) {
            set_error("onng_adjust_path: a pass decided no edge");
            return ONNG_ERR_DEVICE;
        }
        before = h[2];
    }
    ONNG_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tb, kept, out_off, (int)(n + 1), st));
    if (n > 0)
        hipLaunchKernelGGL((pa_compact_kernel<LenT>), dim3(blocks_for(n, 4)), dim3(256), 0, st,
                           g->offsets, out_off, n, g->nbrs, lens, status, out_nb, out_len);
    ONNG_HIP(hipGetLastError());
    ONNG_HIP(hipMemcpyAsync(nnz_out, out_off + n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    ONNG_HIP(hipStreamSynchronize(st));
    return ONNG_OK;
}

onng_status adjust_path_launch(const onng_graph *g, bool int_len, int64_t *offsets,
                               int32_t *nbrs, void *lens, int64_t *nnz_out, void *ws,
                               hipStream_t st) {
    if (int_len)
        return adjust_path_impl<int32_t>(g, offsets, nbrs, static_cast<int32_t *>(lens), nnz_out,
                                         ws, st);
    return adjust_path_impl<float>(g, offsets, nbrs, static_cast<float *>(lens), nnz_out, ws, st);
}

}  // namespace onng
