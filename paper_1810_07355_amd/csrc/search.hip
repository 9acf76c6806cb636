// Batched best-first k-nearest-neighbour search over an adjusted kNN graph:
// KnnSearch (Algorithm 1) of Iwasaki & Miyazaki, one 64-lane wavefront per query.
//
// Per query the wave keeps, in LDS:
//   pool   the best `pool_q` (distance, id) keys seen so far, sorted.  Its first
//          k entries are the result set R of Algorithm 1; r is the k-th
//          distance once k entries exist.  With a rerank, pool_q = pool_factor*k
//          candidates are kept for the exact pass.
//   S      the candidate set, a sorted array [head, size) of keys that are
//          still within the search range; entries that no longer pass
//          d <= r(1+eps) are cut from its tail (they can never be expanded).
//          Keys that do not fit spill to a per-slot global array and come back
//          when the on-chip part runs below their minimum, so S is exact.
//   vis    the visited set C, on chip for a window of consecutive ids around
//          the first seed (one bit per id; the rows are in locality order, so
//          much of a query's neighbourhood falls in it), and a per-slot
//          global bitset (atomic OR) for the other ids.  A query logs every
//          word it turns non-zero and clears those words when it ends, so
//          the bitset is all zero between queries; it is zeroed as a whole
//          only when the workspace's tag says its state is unknown.
//
// One expansion (pop of s, scan of its first e_p edges) is processed as one
// batch: the unvisited neighbours are marked, their distances computed by the
// whole wave, R updated with all of them, then the ones within the updated
// range inserted into S.  Algorithm 1 interleaves these per neighbour; the
// batch gives the same R, visited set, distance count and pop sequence,
// because r never grows: a neighbour Algorithm 1 would insert with an older,
// larger r but the batch rejects is beyond every later range and could only
// end the search when popped, at a pop where the batch's next candidate ends
// it too.
//
// An expansion is one dependent chain, and a query's expansions follow each
// other, so the kernel's time is the sum of these chains over the waves that a
// CU holds (12: registers and LDS), and for a batch that fits the chip, or the
// last queries of a larger one, the longest query's chain itself.  What an
// expansion waits for is kept to one trip to memory, its rows: the offsets,
// adjacency and visited words of the next pop are read ahead (a pop hits them in
// 97 % of the expansions and more).  The rest is instructions: about 600 of
// u8 rows with 4 new rows per expansion, 1,300 of fp8 rows with 68, at 4 cycles
// and more each; so reads are kept in registers or scalars where that saves an
// LDS trip, and a merge of few keys does without searches.
// Kernel alone, before and after that work: u8, 100k x 128, 1000 queries, k 100:
// 935 -> 642 us; f32, 200k x 100, 10k queries: 1511 -> 1253 us; fp8 + rerank,
// 1M x 100, 10k queries: 4300 -> 3177 us.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dist.h"
#include "onng_internal.h"
#include "search_args.h"
#include "wave.h"

namespace onng {

namespace {

constexpr float F_INF = __builtin_inff();

// (1+eps)^2 for squared L2, 1+eps for cosine, rounded to f32; +inf stays +inf.
__device__ __forceinline__ float range_factor(float eps, int metric) {
    if (__builtin_isinf(eps)) return F_INF;
    double t = __dadd_rn(1.0, (double)eps);
    return metric == ONNG_L2SQ ? (float)__dmul_rn(t, t) : (float)t;
}

// Equation 1 for a predicted eps, in f32 (the value used is reported per
// query, so a replay uses the same integer).
__device__ __forceinline__ uint32_t dynamic_ep(float eps, float e0, float we) {
    float v = floorf(exp10f(we * eps) + e0);
    if (!(v < 4294967040.0f)) return 0xffffffffu;
    return v < 1.0f ? 1u : (uint32_t)v;
}

template <int DT, int MT>
struct Q;

// ----------------------------------------------------------- u8, L2^2 ----
template <>
struct Q<ONNG_U8, ONNG_L2SQ> {
    static constexpr int PPL = 2;
    static constexpr bool INT = true;
    u32x4 q[PPL];
    uint32_t qq;
    __device__ __forceinline__ void load(const uint8_t *row, int p, int L, int n16) {
        qq = 0;
#pragma unroll
        for (int t = 0; t < PPL; t++) {
            int pc = p + t * L;
            if (pc < n16) {
                q[t] = load16(row + pc * 16);
                qq += u8_norm_piece(q[t]);
            } else {
                q[t] = u32x4{0, 0, 0, 0};
            }
        }
    }
    // sum over this lane's pieces of (x - q)^2
    __device__ __forceinline__ uint32_t fold(const u32x4 *x, float) const {
        uint32_t s = qq;
#pragma unroll
        for (int t = 0; t < PPL; t++) s += u8_piece(x[t], q[t]);
        return s;
    }
};

// ------------------------------------------------------ float storage ----
template <int DT, int MT>
struct Q {
    static constexpr int PPL = 2;
    static constexpr int N = Piece<DT>::N;
    static constexpr bool INT = false;
    float q[PPL][N];
    // the query is always f32: its piece t of the stored layout covers
    // components [pc*N, pc*N + N)
    __device__ __forceinline__ void load_f32(const float *qrow, int dim, int p, int L, int n16) {
#pragma unroll
        for (int t = 0; t < PPL; t++) {
            int pc = p + t * L;
#pragma unroll
            for (int e = 0; e < N; e++) {
                int c = pc * N + e;
                q[t][e] = (pc < n16 && c < dim) ? qrow[c] : 0.0f;
            }
        }
    }
    // this lane's part of sum (x - q)^2, or of <x, q> for cosine
    __device__ __forceinline__ float fold(const u32x4 *x, float sc) const {
        // two accumulation chains (even / odd components) halve the
        // dependent-FMA latency
        float acc[2] = {0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < PPL; t++) {
            float v[N];
            Piece<DT>::decode(x[t], v);
#pragma unroll
            for (int e = 0; e < N; e++) {
                float xv = v[e];
                // fp8 rows carry a per-row scale: applied per component for
                // L2, once to the dot product for cosine
                if constexpr (DT == ONNG_FP8_E4M3 && MT == ONNG_L2SQ) xv *= sc;
                if constexpr (MT == ONNG_L2SQ) {
                    float df = xv - q[t][e];
                    acc[e & 1] = fmaf(df, df, acc[e & 1]);
                } else {
                    acc[e & 1] = fmaf(xv, q[t][e], acc[e & 1]);
                }
            }
        }
        if constexpr (DT == ONNG_FP8_E4M3 && MT != ONNG_L2SQ) return (acc[0] + acc[1]) * sc;
        return acc[0] + acc[1];
    }
};

template <bool INT>
__device__ __forceinline__ float key_dist(uint64_t key) {
    uint32_t hi = (uint32_t)(key >> 32);
    if constexpr (INT) return (float)hi;
    else return unord_f32(hi);
}

__device__ __forceinline__ float threshold(bool rfull, float r, float f) {
    if (!rfull || __builtin_isinf(f)) return F_INF;
    return __fmul_rn(r, f);
}

struct LdsWave {
    uint64_t *pool;
    uint64_t *S;
    uint64_t *stage;
    uint64_t *stage2;
    uint32_t *ids;
    uint32_t *vis;
    float *misc;
};

// The launch's arguments, read again from the argument segment where they are
// used.  The arguments of the rare parts (set-up, probe phase, output) would
// otherwise be loaded once and kept, and the scalar registers that they then
// take are missing in the expansion loop.
__device__ __forceinline__ const SearchKArgs &late_args() {
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const SearchKArgs *)p;
}

}  // namespace

template <int DT, int MT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3, 8)))
search_kernel(SearchKArgs a0) {
    typedef Q<DT, MT> QT;
    constexpr bool INT = QT::INT;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const SearchKArgs &a = a0;
    const int lane = lane_id();
    const int wib = uni(threadIdx.x / WAVE);   // wave-uniform: derived pointers stay scalar
    const int slot = blockIdx.x * a.waves_per_block + wib;

    char *w = smem + (size_t)wib * a.lds_per_wave;
    LdsWave lds;
    lds.pool = reinterpret_cast<uint64_t *>(w + a.off_pool);
    lds.S = reinterpret_cast<uint64_t *>(w + a.off_s);
    lds.stage = reinterpret_cast<uint64_t *>(w + a.off_stage);
    lds.stage2 = reinterpret_cast<uint64_t *>(w + a.off_stage2);
    lds.ids = reinterpret_cast<uint32_t *>(w + a.off_ids);
    lds.vis = reinterpret_cast<uint32_t *>(w + a.off_vis);
    lds.misc = reinterpret_cast<float *>(w + a.off_misc);
    // 128 keys: the two 64-key stages are adjacent
    uint64_t *const kbuf = lds.stage;

    uint32_t *gbits = a.gbits + (size_t)slot * a.gbits_words;
    int32_t *vlog = a.vlog + (size_t)slot * a.vlog_cap;
    uint64_t *spill0 = a.spill + (size_t)slot * 2 * a.spill_cap;
    // Every launch leaves each slot's bitset all zero (queries clear the words
    // they set).  The workspace tag, written by the last wave of a launch,
    // records the layout that state belongs to; when the caller does not vouch
    // for the workspace or the tag differs, each slot zeroes its bitset first.
    const bool ws_known =
        a.ws_reuse && __hip_atomic_load(a.ws_tag_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                          a.ws_tag;
    if (!ws_known) {
        u32x4 *g4 = reinterpret_cast<u32x4 *>(gbits);
        for (int64_t i = lane; i < a.gbits_words / 4; i += WAVE) g4[i] = u32x4{0, 0, 0, 0};
        __threadfence();
    }

    const int L = a.lanes_per_row;
    const int p = lane & (L - 1);
    const int grp = lane / L;
    const int rpp = WAVE / L;   // rows per pass
    // Lane groups of at least 8, 16, in vector registers, as operands of the sums
    // over a row's lanes.  One- and two-byte rows take 4 or 8 lanes, whose steps
    // beyond are masked (fp8, 1M rows: 3240 -> 3177 us; u8, 100k rows: 654 -> 642);
    // f32 rows mostly take 16, all steps, and keep the branches (1253 us; masked
    // 1284).
    uint32_t g8 = 0u, g16 = 0u;
    if constexpr (DT != ONNG_F32) {
        g8 = L >= 8 ? ~0u : 0u;
        g16 = L >= 16 ? ~0u : 0u;
        asm volatile("" : "+v"(g8), "+v"(g16));
    }
    const uint32_t n_ids = (uint32_t)min(a.n_base, (int64_t)0xFFFFFFFF);
    // byte offsets of this lane's pieces of a row
    int piece[QT::PPL];
    bool has_piece[QT::PPL];
#pragma unroll
    for (int e = 0; e < QT::PPL; e++) {
        has_piece[e] = p + e * L < a.n16;
        piece[e] = min(p + e * L, a.n16 - 1) * 16;
    }
    // row scales: row id's is at scales + id * scale_pitch
    const uint8_t *scales = a.scale_in_row ? a.base + a.base_pitch - 4
                                           : reinterpret_cast<const uint8_t *>(a.base_scale);
    const uint32_t scale_pitch = a.scale_in_row ? (uint32_t)a.base_pitch : 4u;
    // on-chip visited bits: 2^vis_log2 words, one bit per id of a window of
    // W consecutive ids (the rows are in locality order, so a query's
    // neighbourhood has nearby ids); other ids use the global bitset
    const uint32_t W = a.vis_log2 > 0 ? (32u << a.vis_log2) : 0u;

    for (;;) {
        int ticket = 0;
        if (lane == 0) ticket = atomicAdd(a.counter, 1);
        ticket = uni(__shfl(ticket, 0));
        if (ticket >= a.nq) break;
        const int qi = a.order ? uni(a.order[ticket]) : ticket;
        const uint64_t t_start = wall_clock64();

        // ---------------------------------------------- per-query setup --
        const SearchKArgs &as = late_args();
        const int k = as.k_pq ? min(max(uni(as.k_pq[qi]), 1), as.k_stride) : as.k;
        float eps = as.eps_pq ? unif(as.eps_pq[qi]) : as.eps;
        uint32_t ep = as.ep_pq ? uniu(as.ep_pq[qi]) : as.ep;
        if (as.range_from) {
            eps = unif(as.range_from[qi].eps);
            ep = uniu(as.range_from[qi].e_p);
        }
        float cost = eps;
        float f = range_factor(eps, MT);
        if (as.two_phase) {
            f = F_INF;
            ep = as.ep_first;
        }
        const int pool_q = as.has_rr ? min(as.pool_cap, max(k, as.pool_factor * k)) : k;
        int max_dc = as.max_dc_pq ? uni(as.max_dc_pq[qi]) : as.max_dc;
        if (max_dc <= 0) max_dc = INT32_MAX;
        // budget relative to the predicted cost of the chosen range
        auto cost_budget = [&](float c) __attribute__((always_inline)) {
            const float factor = late_args().max_dc_factor;
            if (factor > 0.0f) {
                float b = fminf(factor * c, 2.0e9f);
                max_dc = min(max_dc, max(64, (int)b));
            }
        };
        if (as.range_from) cost_budget(unif(as.range_from[qi].cost));

        QT qr;
        const uint8_t *qrow = a.qry + (size_t)qi * a.q_pitch;
        if constexpr (INT) qr.load(qrow, p, L, a.n16);
        else qr.load_f32(reinterpret_cast<const float *>(qrow), a.dim, p, L, a.n16);

        // state
        int npool = 0;
        int head = 0, size = 0;
        int spill_n = 0, spill_sel = 0;
        uint64_t spill_min = KEY_MAX;
        int log_n = 0;          // words of the global bitset this query made non-zero
        int dc = 0, hops = 0;
        // expansions of the probe phase (0: no such phase)
        const int probe_end = as.two_phase ? (int)as.probe_hops : 0;
        int scanned = 0;   // adjacency entries read (sum of min(deg, e_p) over expansions)
        int flags = 0;
        // search range: f * the k-th distance, infinite until k are known
        float thr = F_INF;
        float r = F_INF;
        bool rfull = false;
        float pruned = __builtin_nanf("");   // range that S was last cut to
        uint64_t plast = KEY_MAX;            // last key of a full pool
        // the first keys of S, one a lane from index front_at on; read again
        // after S has changed
        uint64_t front = KEY_MAX;
        int front_at = 0;
        bool front_ok = false;
        // guessed next expansion (see the expansion loop)
        constexpr uint32_t NO_SPEC = 0xFFFFFFFFu;
        uint32_t spec_id = NO_SPEC;
        int64_t spec_e0 = 0;
        int spec_deg = 0;
        uint32_t spec_nb = 0, spec_nb1 = 0;
        // offsets read ahead: lanes 0 and 1 those of the next pop, lanes 2 and 3
        // those of ofs_id, which is likely to follow it (read with a vector load,
        // which the LDS traffic of the merges does not wait for)
        int64_t ofs = 0;
        uint32_t ofs_id = NO_SPEC;
        // bitset words of the guessed ids, read ahead (first looked at by the
        // guessed expansion: a test beside the read would wait for it there)
        uint32_t spec_wd = 0, spec_wd1 = 0;

        // the on-chip window: W ids around the first seed, within [0, n)
        uint32_t w0 = 0;
        if (W) {
            const int32_t s0 = a.n_seeds > 0 ? a.seeds[(size_t)qi * a.n_seeds] : -1;
            int64_t c = (s0 >= 0 && (int64_t)s0 < a.n_base) ? (int64_t)s0 - (int64_t)(W / 2) : 0;
            const int64_t hi = a.n_base > (int64_t)W ? a.n_base - (int64_t)W : 0;
            c = c < 0 ? 0 : (c > hi ? hi : c);
            w0 = (uint32_t)uni((int)(c & ~31LL));
            for (int i = lane; i < (1 << a.vis_log2); i += WAVE) lds.vis[i] = 0u;
        }
        wave_sync();

        // -------------------------------------------------- helpers ------
        // Ids of two chunks of a list that were found new
        // from words read before them (k0/k1 set) are new in every copy when the
        // list repeats an id.  Keep the first copy in list order (chunk 0
        // before chunk 1, lower lane first), as Algorithm 1's visited set does:
        // a bitmap of 8192 id hashes in LDS finds the lanes whose hash was
        // already taken, and only for those the wave compares ids exactly.
        // The bitmap lives in the distance-key buffer, unused until the batch.
        auto dedupe_known = [&](uint32_t id0, bool &n0, bool k0, uint32_t id1, bool &n1,
                                bool k1) __attribute__((always_inline)) {
            uint32_t *bm = reinterpret_cast<uint32_t *>(kbuf);   // 1 KiB
            reinterpret_cast<u32x4 *>(bm)[lane] = u32x4{0, 0, 0, 0};
            wave_sync();
            bool c0 = false, c1 = false;
            if (k0) {
                const uint32_t h = id0 & 8191u, b = 1u << (h & 31);
                c0 = (atomicOr(&bm[h >> 5], b) & b) != 0u;
            }
            if (k1) {
                const uint32_t h = id1 & 8191u, b = 1u << (h & 31);
                c1 = (atomicOr(&bm[h >> 5], b) & b) != 0u;
            }
            uint64_t cm0 = ballot(c0), cm1 = ballot(c1);
            uint64_t drop0 = 0, drop1 = 0;
            while (cm0 | cm1) {
                uint32_t cid;
                if (cm0) {
                    const int src = (int)__builtin_ctzll(cm0);
                    cm0 &= cm0 - 1;
                    cid = (uint32_t)__builtin_amdgcn_readlane((int)id0, src);
                } else {
                    const int src = (int)__builtin_ctzll(cm1);
                    cm1 &= cm1 - 1;
                    cid = (uint32_t)__builtin_amdgcn_readlane((int)id1, src);
                }
                uint64_t e0 = ballot(k0 && id0 == cid), e1 = ballot(k1 && id1 == cid);
                if (e0) e0 &= e0 - 1;   // the first copy stays new
                else e1 &= e1 - 1;
                drop0 |= e0;
                drop1 |= e1;
            }
            n0 = n0 && !((drop0 >> lane) & 1u);
            n1 = n1 && !((drop1 >> lane) & 1u);
            wave_sync();
        };

        // Mark up to two chunks of ids visited (id1 where two) and list the new
        // ones in lds.ids; returns their number.  `wd` is the bitset word of an
        // id outside the window, read after every earlier mark of the query, so
        // that the mark needs no reply.  Both chunks' marks are under way before
        // either is looked at.
        auto mark = [&](bool v0, uint32_t id0, uint32_t wd0, bool two, bool v1, uint32_t id1,
                        uint32_t wd1) __attribute__((always_inline)) -> int {
            const uint32_t off0 = id0 - w0, off1 = id1 - w0;   // wrap below the window
            const bool in0 = v0 && off0 < W, in1 = v1 && off1 < W;
            uint32_t old0 = 0u, old1 = 0u;
            if (in0) old0 = atomicOr(&lds.vis[off0 >> 5], 1u << (off0 & 31));
            if (in1) old1 = atomicOr(&lds.vis[off1 >> 5], 1u << (off1 & 31));
            // out of the window: the answer came from the word (an id repeated
            // in the list looks new in each copy: see dedupe_known)
            const bool k0 = v0 && !in0 && !(wd0 >> (id0 & 31) & 1u);
            const bool k1 = v1 && !in1 && !(wd1 >> (id1 & 31) & 1u);
            bool n0 = k0 || (in0 && !(old0 >> (off0 & 31) & 1u));
            bool n1 = k1 || (in1 && !(old1 >> (off1 & 31) & 1u));
            if (ballot(k0 || k1)) {
                // set the bits, and log each word that this query turns non-zero
                if (k0)
                    __hip_atomic_fetch_or(&gbits[id0 >> 5], 1u << (id0 & 31), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                if (k1)
                    __hip_atomic_fetch_or(&gbits[id1 >> 5], 1u << (id1 & 31), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                const bool g0 = k0 && wd0 == 0u, g1 = k1 && wd1 == 0u;
                const uint64_t m0 = ballot(g0), m1 = ballot(g1);
                const int at1 = log_n + __popcll(m0);
                if (g0 && log_n + mbcnt(m0) < a.vlog_cap) vlog[log_n + mbcnt(m0)] = (int32_t)(id0 >> 5);
                if (g1 && at1 + mbcnt(m1) < a.vlog_cap) vlog[at1 + mbcnt(m1)] = (int32_t)(id1 >> 5);
                log_n = at1 + __popcll(m1);
                dedupe_known(id0, n0, k0, id1, n1, k1);
            }
            uint64_t m = ballot(n0);
            if (n0) lds.ids[mbcnt(m)] = id0;
            int u = __popcll(m);
            if (two) {
                m = ballot(n1);
                if (n1) lds.ids[u + mbcnt(m)] = id1;
                u += __popcll(m);
            }
            return u;
        };

        // Distances of rows lds.ids[0..u) -> kbuf[i] as keys (u <= 128).  A lane
        // group of L lanes takes one row; NP row passes are requested together.
        // No load sits under a lane mask (a lane without a row or a piece reads
        // the last one again and its piece is cleared before use): masked loads
        // became branches, between which the compiler waited for memory, so
        // that the passes of a batch were served one after the other.
        auto row_passes = [&](auto np_c, int r0, int u) __attribute__((always_inline)) {
            constexpr int NP = decltype(np_c)::value;
            u32x4 x[NP][QT::PPL];
            uint32_t rid[NP];
            float sc[NP];
#pragma unroll
            for (int t = 0; t < NP; t++) rid[t] = lds.ids[min(r0 + t * rpp + grp, u - 1)];
#pragma unroll
            for (int t = 0; t < NP; t++) {
                const uint8_t *rp = a.base + (uint64_t)rid[t] * (uint32_t)a.base_pitch;
#pragma unroll
                for (int e = 0; e < QT::PPL; e++) x[t][e] = load16(rp + piece[e]);
                sc[t] = 1.0f;
                // the row's scale (in its own line when the rows carry it); the
                // lanes of a row read one address
                if constexpr (DT == ONNG_FP8_E4M3)
                    sc[t] = *reinterpret_cast<const float *>(scales + (uint64_t)rid[t] * scale_pitch);
            }
#pragma unroll
            for (int t = 0; t < NP; t++) {
                const int row = r0 + t * rpp + grp;
#pragma unroll
                for (int e = 0; e < QT::PPL; e++) {
                    const uint32_t m = has_piece[e] ? ~0u : 0u;
                    x[t][e] &= u32x4{m, m, m, m};
                }
                // sum over the L lanes of the row (DPP, no LDS round trip)
                typename DistTraits<DT>::acc_t acc = qr.fold(x[t], sc[t]);
                if constexpr (DT == ONNG_F32) acc = group_sum_rt(acc, L);
                else acc = group_sum_masked(acc, L, g8, g16);
                if (row < u && p == 0) {
                    uint32_t dord;
                    if constexpr (INT) dord = acc;
                    else dord = ord_f32(MT == ONNG_COSINE ? 1.0f - acc : acc);
                    kbuf[row] = make_key(dord, rid[t]);
                }
            }
        };
        auto batch_keys = [&](int u) __attribute__((always_inline)) {
            constexpr int MAXP = DT == ONNG_F32 ? 8 : 4;
            for (int r0 = 0; r0 < u; r0 += MAXP * rpp) {
                const int left = u - r0;
                if (MAXP > 4 && left > 4 * rpp) row_passes(std::integral_constant<int, MAXP>(), r0, u);
                else if (left > 2 * rpp) row_passes(std::integral_constant<int, 4>(), r0, u);
                else if (left > rpp) row_passes(std::integral_constant<int, 2>(), r0, u);
                else row_passes(std::integral_constant<int, 1>(), r0, u);
            }
            wave_sync();
        };

        // spill a key that fell past the on-chip capacity of S; spilled keys
        // arrive in ascending order, so index 0 is the smallest of this merge
        uint64_t first_spilled = KEY_MAX;
        auto spill_put = [&](int idx, uint64_t key) __attribute__((always_inline)) {
            int pos = spill_n + idx;
            if (idx == 0) first_spilled = key;
            if (pos < a.spill_cap) spill0[(size_t)spill_sel * a.spill_cap + pos] = key;
        };

        // Merge sorted batch (lane j < nb holds j-th key) into S.
        auto s_insert = [&](uint64_t key, int nb) __attribute__((always_inline)) {
            if (nb == 0) return;
            front_ok = false;
            if (size + nb > a.s_cap && head > 0) {
                // compact the live part to the front
                int live = size - head;
                for (int c0 = 0; c0 < live; c0 += WAVE) {
                    uint64_t v = 0;
                    if (c0 + lane < live) v = lds.S[head + c0 + lane];
                    wave_sync();
                    if (c0 + lane < live) lds.S[c0 + lane] = v;
                    wave_sync();
                }
                size = live;
                head = 0;
            }
            first_spilled = KEY_MAX;
            int total = merge_sorted(lds.S, head, size - head, key, nb, a.s_cap - head, lds.stage,
                                     spill_put);
            int over = total - (a.s_cap - head);
            if (over > 0) {
                uint64_t mn = first_spilled;
                for (int m = 32; m >= 1; m >>= 1) {
                    uint64_t o = shfl_xor64(mn, m);
                    mn = o < mn ? o : mn;
                }
                mn = uni64(mn);
                spill_min = mn < spill_min ? mn : spill_min;
                if (spill_n + over > a.spill_cap) flags |= ONNG_QF_CAPACITY;
                spill_n = min(spill_n + over, (int)a.spill_cap);
                flags |= ONNG_QF_SPILLED;
                size = a.s_cap;
            } else {
                size = head + total;
            }
        };

        // Drop S entries beyond the range (a suffix of the sorted array).
        auto s_prune = [&]() __attribute__((always_inline)) {
            if (thr == pruned || size == head || __builtin_isinf(thr)) return;
            pruned = thr;
            if (key_dist<INT>(lds.S[size - 1]) <= thr) return;   // all within range
            // first index with d > thr: every stride-th entry first, then the
            // entries between the last sample within range and the next one
            const int n = size - head;
            const int stride = (n + WAVE - 1) / WAVE;
            const int i1 = head + lane * stride;
            uint64_t m = ballot(i1 < size && key_dist<INT>(lds.S[i1]) > thr);
            const int ns = (n + stride - 1) / stride;
            const int b = m ? (int)__builtin_ctzll(m) : ns;
            if (b == 0) {
                size = head;
                return;
            }
            const int lo = head + (b - 1) * stride + 1;
            const int hi = min(head + b * stride, size);
            int cut = hi;
            for (int c = lo; c < hi; c += WAVE) {
                const int i2 = c + lane;
                uint64_t m2 = ballot(i2 < hi && key_dist<INT>(lds.S[i2]) > thr);
                if (m2) {
                    cut = c + (int)__builtin_ctzll(m2);
                    break;
                }
            }
            size = uni(cut);
        };

        // Merge sorted keys into the pool (R and rerank candidates).
        auto pool_insert = [&](uint64_t key, int nb) __attribute__((always_inline)) {
            // a full pool only takes keys below its last one (a sorted prefix)
            nb = __popcll(ballot(lane < nb && key < plast));
            if (nb == 0) return;
            int total = merge_sorted(lds.pool, 0, npool, key, nb, pool_q, lds.stage, NoSpill());
            npool = min(total, pool_q);
            const uint64_t pk = lds.pool[k - 1], pl = lds.pool[pool_q - 1];
            if (npool >= k) {
                rfull = true;
                r = unif(key_dist<INT>(pk));
                thr = unif(threshold(true, r, f));
            }
            if (npool == pool_q) plast = uni64(pl);
        };

        // Process a sorted batch: R first (absorb_pool), then the range test
        // with the new r and the insertion into S (absorb_s).
        auto absorb_pool = [&](uint64_t key, int u) __attribute__((always_inline)) { pool_insert(key, u); };
        auto absorb_s = [&](uint64_t key, int u, bool to_s) __attribute__((always_inline)) {
            // the batch is sorted, so the keys within range are a prefix
            bool keep = lane < u && key_dist<INT>(key) <= thr;
            if (!to_s) keep = lane < u;
            const int nk = __popcll(ballot(keep));
            const uint64_t ck = lane < nk ? key : KEY_MAX;
            s_prune();
            if (!to_s) pruned = __builtin_nanf("");   // taken without the range test
            s_insert(ck, nk);
        };
        auto absorb = [&](uint64_t key, int u, bool to_s) __attribute__((always_inline)) {
            absorb_pool(key, u);
            absorb_s(key, u, to_s);
        };

        // Bring spilled keys back: merge every live spilled key into S, the
        // ones that do not fit go to the other spill buffer.
        auto refill = [&]() __attribute__((always_inline)) {
            __threadfence_block();   // spilled keys were stored by other lanes
            front_ok = false;
            int n_old = spill_n;
            int sel_old = spill_sel;
            spill_sel ^= 1;
            spill_n = 0;
            spill_min = KEY_MAX;
            for (int c0 = 0; c0 < n_old; c0 += WAVE) {
                uint64_t v = KEY_MAX;
                if (c0 + lane < n_old) {
                    v = spill0[(size_t)sel_old * a.spill_cap + c0 + lane];
                    if (key_dist<INT>(v) > thr) v = KEY_MAX;   // dead
                }
                uint64_t m = ballot(v != KEY_MAX);
                int nb = __popcll(m);
                if (nb == 0) continue;
                v = wave_sort(v, WAVE);
                s_prune();
                s_insert(v, nb);
            }
        };

        // ------------------------------------------------------ seeds ----
        {
            bool valid = false;
            uint32_t sid = 0;
            if (lane < a.n_seeds) {
                int32_t s = a.seeds[(size_t)qi * a.n_seeds + lane];
                valid = s >= 0 && (int64_t)s < a.n_base;
                sid = valid ? (uint32_t)s : 0u;
            }
            // nothing is marked yet: every word is known to be zero
            const int u = mark(valid, sid, 0u, false, false, 0u, 0u);
            wave_sync();
            batch_keys(u);
            dc += u;
            uint64_t key = lane < u ? kbuf[lane] : KEY_MAX;
            wave_sync();
            key = wave_sort(key, pow2_at_least(u));
            if (probe_end > 0) lds.misc[lane] = lane < u ? key_dist<INT>(key) : 0.0f;
            if (probe_end > 0 && lane == 0) lds.misc[64] = (float)u;
            // every seed enters S (no range test) and is offered to R
            absorb(key, u, false);
        }

        // ------------------------------------------------- main loop -----
        // One pass is up to two 64-edge chunks of the expanded node: their ids
        // and visited marks, then one distance batch for the new nodes.  A
        // longer list takes more passes (g0 is the pass's first edge).
        int np = 0, g0 = 0;
        int64_t e0 = 0;
        for (;;) {
            const bool pop = g0 >= np;
            if (pop) {
                if (head == size && spill_n == 0) break;              // S empty
                if (dc >= max_dc) {                                   // budget spent
                    flags |= ONNG_QF_BUDGET;
                    break;
                }
                if (spill_n > 0 && (head == size || uni64(lds.S[head]) > spill_min)) {
                    refill();
                    if (head == size) break;
                }
            }
            // the pop and the two keys behind it
            if (!front_ok || head - front_at > WAVE - 4) {
                front = lds.S[max(min(head + lane, size - 1), 0)];
                front_at = head;
                front_ok = true;
            }
            bool hit = false;
            if (pop) {
                const uint64_t sk = readlane64(front, head - front_at);
                head++;
                if (key_dist<INT>(sk) > thr) break;                   // d(s,q) > r(1+eps)
                hops++;
                const uint32_t s = (uint32_t)sk;
                // adjacency of s: read ahead when the previous expansion
                // guessed this pop, else read now
                hit = s == spec_id;
                int deg;
                if (hit) {
                    e0 = spec_e0;
                    deg = spec_deg;
                } else {
                    e0 = a.offsets[s];
                    deg = (int)(a.offsets[s + 1] - e0);
                }
                np = (int)min(ep, (uint32_t)deg);
                g0 = 0;
                scanned += np;
            }
            spec_id = NO_SPEC;
            const int left = np - g0;
            const bool last = left <= 2 * WAVE;
            const uint64_t head_key = head < size ? readlane64(front, head - front_at) : KEY_MAX;
            const uint32_t next1 = (uint32_t)head_key;   // NO_SPEC where S is empty
            const uint32_t next2 = head + 1 < size ? (uint32_t)readlane64(front, head + 1 - front_at)
                                                   : NO_SPEC;
            // The next pop is next1 unless this expansion finds a nearer node
            // (at the measured settings next1 it is in 62 to 94 % of the
            // expansions), so its reads start now: the offsets of next1 and of
            // next2 are requested here, and where next1 was next2 one
            // expansion ago its offsets are known and the adjacency itself is
            // requested before this expansion's rows.
            const bool ahead = next1 != NO_SPEC && next1 == ofs_id;
            int64_t n_e0 = readlane64(ofs, 2);
            int n_deg = (int)(readlane64(ofs, 3) - n_e0);
            // What was read ahead has to be there from here on, a wrong guess
            // too: else the compiler, which does not see that these loads are
            // over, waits for all loads in flight where their registers are
            // written next, in the middle of the expansion.
            asm volatile("" : "+v"(spec_nb), "+v"(spec_nb1), "+v"(spec_wd), "+v"(spec_wd1));
            // The reads below are masked per lane and write their registers in
            // place; lanes without a value keep an old one, which nothing looks
            // at.  Under a branch of the whole wave (or with zeros for those
            // lanes) the registers would be copied where the paths join, and a
            // copy waits for the load.
            int nl0 = 0, nl1 = 0;
            auto read_adjacency = [&](bool go, int64_t first, int n) __attribute__((always_inline)) {
                if (!go) return;
                nl0 = min(n, WAVE);
                nl1 = min(n - nl0, WAVE);
                if (lane < nl0) spec_nb = (uint32_t)a.nbrs[first + lane];
                if (lane < nl1) spec_nb1 = (uint32_t)a.nbrs[first + WAVE + lane];
            };
            auto read_visited = [&](bool go) __attribute__((always_inline)) {
                if (!go) return;
                // every earlier mark is complete before the visited words are
                // read (of ids outside the window: the others are on chip)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                const bool c0 = (lane < nl0) & (spec_nb < n_ids) & (spec_nb - w0 >= W);
                const bool c1 = (lane < nl1) & (spec_nb1 < n_ids) & (spec_nb1 - w0 >= W);
                if (c0)
                    spec_wd = __hip_atomic_load(&gbits[spec_nb >> 5], __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
                if (c1)
                    spec_wd1 = __hip_atomic_load(&gbits[spec_nb1 >> 5], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            };
            read_adjacency(!hit, e0 + g0, left);
            read_visited(!hit);
            {
                const uint32_t id = (lane & 2) ? next2 : next1;
                ofs = a.offsets[(size_t)(id != NO_SPEC ? id : 0u) + (lane & 1)];
                ofs_id = next2;
            }
            const int u = mark(lane < left && spec_nb < n_ids, spec_nb, spec_wd, WAVE < left,
                               WAVE + lane < left && spec_nb1 < n_ids, spec_nb1, spec_wd1);
            // the guess's reads: 0 nothing usable, 1 offsets requested,
            // 2 adjacency requested, 3 visited words requested
            int stage = 0;
            auto guess_adjacency = [&](bool go, int64_t first, int n) __attribute__((always_inline)) {
                read_adjacency(go, first, n);
                spec_e0 = go ? first : spec_e0;
                spec_deg = go ? n : spec_deg;
                stage = go ? 2 : stage;
            };
            auto guess_visited = [&]() __attribute__((always_inline)) {
                read_visited(stage == 2);
                stage = stage == 2 ? 3 : stage;
            };
            guess_adjacency(last && ahead, n_e0, n_deg);
            uint64_t k0 = KEY_MAX, k1 = KEY_MAX;
            int nk = 0;
            if (u > 0) {
                wave_sync();
                batch_keys(u);
                dc += u;
                k0 = lane < u ? kbuf[lane] : KEY_MAX;
                k1 = lane + WAVE < u ? kbuf[lane + WAVE] : KEY_MAX;
                wave_sync();
            }
            guess_visited();
            // Keys that can neither enter S (beyond the current range,
            // which only shrinks) nor the pool (beyond its last key when
            // full) are dropped before sorting.
            if (u > 0) {
                bool keep0 = lane < u && (key_dist<INT>(k0) <= thr || k0 < plast);
                bool keep1 = lane + WAVE < u && (key_dist<INT>(k1) <= thr || k1 < plast);
                uint64_t m0 = ballot(keep0), m1 = ballot(keep1);
                const int n0 = __popcll(m0);
                nk = n0 + __popcll(m1);
                if (nk < u && nk > 0) {
                    if (keep0) kbuf[mbcnt(m0)] = k0;
                    if (keep1) kbuf[n0 + mbcnt(m1)] = k1;
                    wave_sync();
                    k0 = lane < nk ? kbuf[lane] : KEY_MAX;
                    k1 = lane + WAVE < nk ? kbuf[lane + WAVE] : KEY_MAX;
                    wave_sync();
                }
            }
            const int na = min(nk, WAVE), nb2 = nk - na;
            if (na > 0) k0 = wave_sort(k0, pow2_at_least(na));
            if (nb2 > 0) k1 = wave_sort(k1, pow2_at_least(nb2));
            // Guess the next pop (the smaller of S's head and this group's
            // minimum, when within range and no spilled key is smaller).
            // Where it is next1 its reads are under way; else they start
            // here, a dependent chain (offsets, adjacency, visited words)
            // of which each step is issued one merge after the previous
            // one, so that its latency overlaps the merge.  A wrong guess
            // only wastes the reads.
            bool have_ofs = false;
            if (last) {
                uint64_t cand = head_key;
                if (na > 0) {
                    const uint64_t b0 = readlane64(k0, 0);
                    cand = b0 < cand ? b0 : cand;
                }
                if (nb2 > 0) {
                    const uint64_t b1 = readlane64(k1, 0);
                    cand = b1 < cand ? b1 : cand;
                }
                if (cand != KEY_MAX && !(spill_n > 0 && spill_min < cand) &&
                    key_dist<INT>(cand) <= thr) {
                    spec_id = (uint32_t)cand;
                    if (spec_id != next1) {
                        stage = 1;
                        ofs_id = next1;   // what then follows it
                    } else if (stage == 0) {
                        stage = 1;        // requested at the pop
                        have_ofs = true;
                    }
                } else {
                    stage = 0;
                }
            }
            {
                const uint32_t id = (lane & 2) && next1 != NO_SPEC ? next1 : spec_id;
                if (lane < (stage == 1 && !have_ofs ? WAVE : 0)) ofs = a.offsets[(size_t)id + (lane & 1)];
            }
            if (na > 0) absorb_pool(k0, na);
            if (stage == 1) {
                n_e0 = readlane64(ofs, 0);
                n_deg = (int)(readlane64(ofs, 1) - n_e0);
            }
            guess_adjacency(stage == 1, n_e0, n_deg);
            if (na > 0) absorb_s(k0, na, true);
            guess_visited();
            if (nb2 > 0) absorb(k1, nb2, true);
            g0 += 2 * WAVE;
            if (!last) continue;

            if (probe_end > 0 && hops == probe_end) {
                const SearchKArgs &ap = late_args();
                // ---- state after the probe expansions -> search range ----
                if (spill_n > 0) refill();   // the smallest keys of S on chip
                int nseed = (int)lds.misc[64];
                int ns = size - head + spill_n;
                int m = min(size - head, 64);
                float rmax = npool > 0 ? key_dist<INT>(lds.pool[min(npool, k) - 1]) : 0.0f;
                // lane t < 14 computes feature t
                float fv = 0.0f;
                if (lane < 8) fv = nseed == 0 ? 0.0f : lds.misc[lane < nseed ? lane : nseed - 1];
                else if (lane == 8) fv = (float)ns;
                else if (lane == 9) fv = m > 0 ? key_dist<INT>(lds.S[head]) : rmax;
                else if (lane == 10) fv = m > 0 ? key_dist<INT>(lds.S[head + (m + 1) / 2 - 1]) : rmax;
                else if (lane == 11) fv = m > 0 ? key_dist<INT>(lds.S[head + m - 1]) : rmax;
                else if (lane == 12) fv = rmax;
                else if (lane == 13) fv = (float)dc;
                if (ap.feat_out && lane < ONNG_NFEAT) ap.feat_out[(size_t)qi * ONNG_NFEAT + lane] = fv;
                if (ap.has_pred) {
                    eps = predict_eps(ap.pred, fv, MT, qi, lane, lds.misc + 72, &cost);
                    eps = unif(eps);
                    cost = unif(cost);
                    if (ap.pred.mode == ONNG_PRED_CURVE) cost_budget(cost);
                    ep = ap.pred.we >= 0.0f ? dynamic_ep(eps, ap.pred.e0, ap.pred.we)
                                           : (ap.ep_pq ? uniu(ap.ep_pq[qi]) : ap.ep);
                } else {
                    eps = ap.eps_pq ? unif(ap.eps_pq[qi]) : ap.eps;
                    ep = ap.ep_pq ? uniu(ap.ep_pq[qi]) : ap.ep;
                }
                f = range_factor(eps, MT);
                thr = unif(threshold(rfull, r, f));
                s_prune();
                if (ap.predict_only) break;   // the range is all this pass reports
            }
        }

        // ---------------------------------------------- rerank, output ---
        const SearchKArgs &ao = late_args();
        int nout = min(npool, k);
        if (ao.predict_only) {
            // no result rows in a predict-only pass
        } else if (ao.has_rr && npool > 0) {
            // exact f32 distances of the pool from the f32 rows
            for (int c0 = 0; c0 < npool; c0 += WAVE) {
                if (c0 + lane < npool) lds.ids[lane] = (uint32_t)lds.pool[c0 + lane];
                wave_sync();
                int u = min(WAVE, npool - c0);
                // 16 rows per pass, 4 lanes per row; a lane reads 16-byte
                // pieces pp, pp + 4, ... of its row, up to 8 at once, so that a
                // pass waits for memory once (rows of up to 128 components)
                const int pp = lane & 3;
                const int n4 = (ao.dim + 3) >> 2;
                const float4 *qf4 = reinterpret_cast<const float4 *>(qrow);
                for (int r0 = 0; r0 < u; r0 += 16) {
                    const int row = r0 + (lane >> 2);
                    const bool rv = row < u;
                    const uint32_t id = rv ? lds.ids[row] : 0u;
                    const float4 *xr4 =
                        reinterpret_cast<const float4 *>(ao.rr_base + (size_t)id * ao.rr_pitch);
                    float acc = 0.0f;
                    for (int j0 = 0; j0 < n4; j0 += 32) {
                        float4 xv[8], qv[8];
#pragma unroll
                        for (int t = 0; t < 8; t++) {
                            const int c4 = j0 + pp + 4 * t;
                            const bool in = rv && c4 < n4;
                            xv[t] = in ? xr4[c4] : float4{0.0f, 0.0f, 0.0f, 0.0f};
                            qv[t] = in ? qf4[c4] : float4{0.0f, 0.0f, 0.0f, 0.0f};
                        }
#pragma unroll
                        for (int t = 0; t < 8; t++) {
                            const int c = 4 * (j0 + pp + 4 * t);
                            const float xs[4] = {xv[t].x, xv[t].y, xv[t].z, xv[t].w};
                            const float qs[4] = {qv[t].x, qv[t].y, qv[t].z, qv[t].w};
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                // components past dim (a row's padding) count as zero
                                const float xe = c + e < ao.dim ? xs[e] : 0.0f;
                                const float qe = c + e < ao.dim ? qs[e] : 0.0f;
                                if constexpr (MT == ONNG_L2SQ) {
                                    const float df = xe - qe;
                                    acc = fmaf(df, df, acc);
                                } else {
                                    acc = fmaf(xe, qe, acc);
                                }
                            }
                        }
                    }
                    acc += __shfl_xor(acc, 1);
                    acc += __shfl_xor(acc, 2);
                    if (rv && pp == 0) {
                        float d = MT == ONNG_COSINE ? 1.0f - acc : acc;
                        lds.stage2[row] = make_key(ord_f32(d), id);
                    }
                }
                wave_sync();
                uint64_t key = lane < u ? lds.stage2[lane] : KEY_MAX;
                wave_sync();
                key = wave_sort(key, pow2_at_least(u));
                // reuse S as the top-k accumulator of the reranked keys
                int cur = c0 == 0 ? 0 : min(c0, k);
                merge_sorted(lds.S, 0, cur, key, u, k, lds.stage, NoSpill());
            }
            nout = min(npool, k);
            for (int i = lane; i < ao.k_stride; i += WAVE) {
                int32_t id = -1;
                float d = F_INF;
                if (i < nout) {
                    uint64_t key = lds.S[i];
                    id = (int32_t)(uint32_t)key;
                    d = unord_f32((uint32_t)(key >> 32));
                    if (ao.id_map) id = ao.id_map[id];
                }
                ao.out_ids[(size_t)qi * ao.k_stride + i] = id;
                reinterpret_cast<float *>(ao.out_d)[(size_t)qi * ao.k_stride + i] = d;
            }
        } else {
            for (int i = lane; i < ao.k_stride; i += WAVE) {
                int32_t id = -1;
                uint64_t key = i < nout ? lds.pool[i] : KEY_MAX;
                if (i < nout) id = (int32_t)(uint32_t)key;
                if (i < nout && ao.id_map) id = ao.id_map[id];
                ao.out_ids[(size_t)qi * ao.k_stride + i] = id;
                if constexpr (INT) {
                    reinterpret_cast<int32_t *>(ao.out_d)[(size_t)qi * ao.k_stride + i] =
                        i < nout ? (int32_t)(key >> 32) : INT32_MAX;
                } else {
                    reinterpret_cast<float *>(ao.out_d)[(size_t)qi * ao.k_stride + i] =
                        i < nout ? unord_f32((uint32_t)(key >> 32)) : F_INF;
                }
            }
        }
        if (nout < k && !ao.predict_only) flags |= ONNG_QF_PADDED;
        if (lane == 0) {
            onng_query_stats st;
            st.dc = dc;
            st.hops = hops;
            st.flags = flags;
            st.e_p = ep;
            st.eps = eps;
            st.scanned = scanned;
            st.cost = cost;
            st.us = (float)(wall_clock64() - t_start) * ao.us_per_tick;
            ao.stats[qi] = st;
        }

        // leave the global visited bitset clean for the next query
        if (log_n > 0) {
            __threadfence_block();   // the log was written by other lanes
            if (log_n <= a.vlog_cap) {
                // eight log entries per lane in flight, then their stores
                for (int i0 = 0; i0 < log_n; i0 += 8 * WAVE) {
                    int32_t wd[8];
#pragma unroll
                    for (int t = 0; t < 8; t++) {
                        const int i = i0 + t * WAVE + lane;
                        wd[t] = i < log_n ? vlog[i] : -1;
                    }
#pragma unroll
                    for (int t = 0; t < 8; t++)
                        if (wd[t] >= 0) gbits[(uint32_t)wd[t]] = 0u;
                }
            } else {
                u32x4 *g4 = reinterpret_cast<u32x4 *>(gbits);
                for (int64_t i = lane; i < a.gbits_words / 4; i += WAVE) g4[i] = u32x4{0, 0, 0, 0};
            }
            __threadfence_block();
        }
        wave_sync();
    }

    // The last wave of the launch records the layout whose bitsets are now
    // all zero.
    if (lane == 0) {
        __threadfence();
        const int total = (int)gridDim.x * a.waves_per_block;
        if (atomicAdd(a.counter + 1, 1) == total - 1)
            __hip_atomic_store(a.ws_tag_at, a.ws_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Dispatch -----------------------------------------------------------------

#define ONNG_SEARCH_INST(DT, MT)                                                      \
    template __global__ void search_kernel<DT, MT>(SearchKArgs);

ONNG_SEARCH_INST(ONNG_U8, ONNG_L2SQ)
ONNG_SEARCH_INST(ONNG_F32, ONNG_L2SQ)
ONNG_SEARCH_INST(ONNG_F32, ONNG_COSINE)
ONNG_SEARCH_INST(ONNG_F16, ONNG_L2SQ)
ONNG_SEARCH_INST(ONNG_F16, ONNG_COSINE)
ONNG_SEARCH_INST(ONNG_BF16, ONNG_L2SQ)
ONNG_SEARCH_INST(ONNG_BF16, ONNG_COSINE)
ONNG_SEARCH_INST(ONNG_FP8_E4M3, ONNG_L2SQ)
ONNG_SEARCH_INST(ONNG_FP8_E4M3, ONNG_COSINE)

// work ticket (c[0]) and finished-wave count (c[1]) of a search launch
__global__ void reset_counter_kernel(int32_t *c) {
    c[0] = 0;
    c[1] = 0;
}

const void *search_kernel_ptr(int dtype, int metric) {
    switch (dtype) {
    case ONNG_U8: return metric == ONNG_L2SQ ? (const void *)search_kernel<ONNG_U8, ONNG_L2SQ> : nullptr;
    case ONNG_F32:
        return metric == ONNG_L2SQ ? (const void *)search_kernel<ONNG_F32, ONNG_L2SQ>
                                   : (const void *)search_kernel<ONNG_F32, ONNG_COSINE>;
    case ONNG_F16:
        return metric == ONNG_L2SQ ? (const void *)search_kernel<ONNG_F16, ONNG_L2SQ>
                                   : (const void *)search_kernel<ONNG_F16, ONNG_COSINE>;
    case ONNG_BF16:
        return metric == ONNG_L2SQ ? (const void *)search_kernel<ONNG_BF16, ONNG_L2SQ>
                                   : (const void *)search_kernel<ONNG_BF16, ONNG_COSINE>;
    case ONNG_FP8_E4M3:
        return metric == ONNG_L2SQ ? (const void *)search_kernel<ONNG_FP8_E4M3, ONNG_L2SQ>
                                   : (const void *)search_kernel<ONNG_FP8_E4M3, ONNG_COSINE>;
    }
    return nullptr;
}

// forget the workspace tag, so that the next launch zeroes the bitsets
__global__ void clear_tag_kernel(uint64_t *tag) { *tag = 0; }

const void *reset_counter_kernel_ptr() { return (const void *)reset_counter_kernel; }
const void *clear_tag_kernel_ptr() { return (const void *)clear_tag_kernel; }

}  // namespace onng
