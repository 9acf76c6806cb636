// Exact top-k in two passes over the distance matrix: a bound, then a filter.
//
//  bound   Distances of a sample of the base rows, a power of two spread over
//          all of them.  Each lane keeps the smallest distance of a group of
//          columns (a few of each tile, over several tiles), and per query row
//          the rank-th smallest group minimum is at least the row's k-th
//          smallest distance: the minima belong to distinct base rows.
//  filter  All distances; the few (about k / sampled share) that do not exceed
//          the bound go to the row's candidate buffer.
//
// One wave per row then sorts its candidates.  Neither pass keeps lists, so
// the LDS holds a tile and a short candidate queue per wave, several blocks
// share a compute unit instead of one, and the matrix instructions are what is
// left to wait for.  The products are those of topk.hip, in the same order: the distances
// are the same bit for bit.  A row whose buffer overflows (distances tied or
// very unevenly spread), or holds fewer than k, is left to topk_kernel, which
// redoes such rows only.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "onng_internal.h"
#include "topk_common.h"
#include "wave.h"

namespace onng {
namespace topk_detail {

constexpr int BOUND_QUEUE = 192;          // candidates a wave holds before it places them
constexpr int64_t BOUND_CHUNK = 65536;    // query rows whose candidates are held at a time

struct BoundArgs {
    TopkArgs t;               // nq: end of the chunk's query rows
    int64_t row_first;        // first query row of the chunk; the buffers below are the chunk's
    int32_t ns_log2;          // sampled rows (bound)
    int32_t group_tiles;      // tiles a lane's minimum runs over (bound)
    int32_t quads;            // the minima of four lanes make one group (bound)
    int32_t groups;           // minima per query row
    uint32_t *mins;           // [rows][groups]
    const uint32_t *tau;      // [rows] distances below it pass (filter)
    int32_t *cnt;             // [rows] candidates found (may exceed cap)
    uint64_t *cand;           // [rows][cap]
    int32_t cap;
};

// waves, LDS bytes of a block whose query rows take RW waves (16 rows each);
// with one, four waves share the 16 rows and split the tile's columns
constexpr int bound_threads(int rw) { return rw == 8 ? 512 : 256; }
inline size_t bound_lds(int lds_pitch, int rw, bool filter) {
    return (size_t)2 * BN * (lds_pitch + 8) +
           (filter ? (size_t)bound_threads(rw) / WAVE * (BOUND_QUEUE * 10 + 64) : 0);
}

// A block: RW waves with 16 query rows each, over all 64 columns of a tile; for
// RW = 1 (at most 16 rows in all) four waves, each with one of a tile's four
// 16-column blocks.
template <int DT, int MT, int NCH, int RW, bool BOUND>
__global__ void __launch_bounds__(bound_threads(RW), NCH <= 8 ? (RW == 4 ? 3 : 4) : 2) topk_bound_kernel(BoundArgs A) {
    constexpr bool U8 = DT == ONNG_U8;
    constexpr int KQ = 4 * NCH;
    constexpr int NCB = RW == 1 ? 1 : 4;
    constexpr int CW = 4 / NCB;
    constexpr int CPR = NCH * 4;         // 16-byte chunks of a staged row
    constexpr int total = BN * CPR;
    constexpr int nthr = bound_threads(RW);
    constexpr int STG = (total + nthr - 1) / nthr;   // chunks per thread
    constexpr int bm = RW * 16;
    const TopkArgs &a = A.t;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int wv = uni(threadIdx.x / WAVE);
    const int rw = RW == 1 ? 0 : wv, cw = RW == 1 ? wv : 0;
    const int64_t lrow0 = (int64_t)blockIdx.x * bm;   // within the chunk
    const int64_t row0 = A.row_first + lrow0;
    constexpr bool norms = U8 || MT == ONNG_L2SQ;

    // LDS: two of [B tile][norms BN][ids BN] (the next tile is stored while
    // this one may still be read: one barrier a tile), filter: per wave [queue
    // keys][counts 16][queue rows][numbers]
    const uint32_t buf_bytes = BN * ((uint32_t)a.lds_pitch + 8u);
    char *wq = smem + 2 * buf_bytes + (size_t)wv * (BOUND_QUEUE * 10 + 64);
    uint64_t *q_key = reinterpret_cast<uint64_t *>(wq);
    int32_t *q_cnt = reinterpret_cast<int32_t *>(q_key + BOUND_QUEUE);
    uint8_t *q_row = reinterpret_cast<uint8_t *>(q_cnt + 16);
    uint8_t *q_num = q_row + BOUND_QUEUE;   // number within its row
    int qn_held = 0;

    // ---- this wave's 16 query rows as MFMA A operands ----
    const int arow = lane & 15;
    const int kg = lane >> 4;
    const int64_t qrow = row0 + rw * 16 + arow;
    const bool qvalid = qrow < a.nq;
    const uint8_t *qp = a.q + (qvalid ? qrow : 0) * a.q_pitch;
    i32x4 A8[U8 ? NCH : 1];
    float AF[U8 ? 1 : KQ];
    if constexpr (U8) {
#pragma unroll
        for (int s = 0; s < NCH; s++)
            A8[s] = qvalid ? shifted16(qp, s * 64 + kg * 16, a.dim) : i32x4{0, 0, 0, 0};
    } else {
        const float *qf = reinterpret_cast<const float *>(qp);
#pragma unroll
        for (int s = 0; s < KQ; s++) {
            const int c = kg * KQ + s;
            AF[s] = (qvalid && c < a.dim) ? qf[c] : 0.0f;
        }
    }
    // the 4 output rows this lane sees in C (rows 4*kg + r)
    int32_t qn8[4] = {0, 0, 0, 0};
    float qnf[4] = {0, 0, 0, 0};
    uint32_t tau[4] = {0, 0, 0, 0};
    bool rok[4];
    const int64_t lcrow0 = lrow0 + rw * 16 + 4 * kg, crow0 = A.row_first + lcrow0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        rok[r] = crow0 + r < a.nq;
        if (rok[r]) {
            if constexpr (U8) qn8[r] = reinterpret_cast<const int32_t *>(a.qn)[crow0 + r];
            else if constexpr (MT == ONNG_L2SQ) qnf[r] = reinterpret_cast<const float *>(a.qn)[crow0 + r];
            if (!BOUND) tau[r] = A.tau[lcrow0 + r];
        }
    }
    const bool live = row0 + rw * 16 < a.nq;
    bool any_passes = false;   // of the block's rows, the same in every wave
    if constexpr (!BOUND) {
        uint32_t t = 0;
        for (int i = lane; i < bm; i += WAVE)
            if (row0 + i < a.nq) t |= A.tau[lrow0 + i];
        any_passes = ballot(t != 0) != 0;
    }

    const int ntiles = BOUND ? (1 << A.ns_log2) / BN : (int)((a.nb + BN - 1) / BN);
    const int t_beg = blockIdx.y * a.tiles_per_split;
    const int t_end = min(ntiles, t_beg + a.tiles_per_split);
    const uint32_t bp32 = (uint32_t)a.b_pitch;
    const int cmax = (int)min<int64_t>(CPR, a.b_pitch / 16);   // chunks a global row holds

    // the next tile's rows are read into registers while the current one is computed
    uint4 stg[STG];
    uint32_t side_g = 0;
    auto fetch_tile = [&](int t) {
        const int64_t c0 = (int64_t)t * BN;
        const int rows = BOUND ? BN : (int)min<int64_t>(BN, a.nb - c0);
        const uint8_t *tb = a.b + c0 * a.b_pitch;
        auto at = [&](int r, int c) {
            if (BOUND)
                return reinterpret_cast<const uint4 *>(
                    a.b + sample_row((uint32_t)(c0 + r), A.ns_log2, a.nb) * a.b_pitch + (uint32_t)c * 16u);
            return reinterpret_cast<const uint4 *>(tb + ((uint32_t)r * bp32 + (uint32_t)c * 16u));
        };
        if (rows == BN && cmax == CPR) {
#pragma unroll
            for (int j = 0; j < STG; j++) {
                const int i = threadIdx.x + j * nthr;
                if (total % nthr == 0 || i < total) stg[j] = *at(i / CPR, i % CPR);
            }
        } else {
#pragma unroll
            for (int j = 0; j < STG; j++) {
                const int i = threadIdx.x + j * nthr;
                const int r = i / CPR, c = i - r * CPR;
                stg[j] = uint4{0, 0, 0, 0};
                if (i < total && r < rows && c < cmax) stg[j] = *at(r, c);
            }
        }
        if (!BOUND && a.b_ids && threadIdx.x < BN)
            side_g = threadIdx.x < rows ? (uint32_t)a.b_ids[c0 + threadIdx.x] : 0u;
    };
    // the fetched rows into a buffer; components at or past dim become 0 (a
    // row's padding may hold anything)
    auto put_tile = [&](uint8_t *buf) {
#pragma unroll
        for (int j = 0; j < STG; j++) {
            const int i = threadIdx.x + j * nthr;
            if (i >= total) continue;
            const int r = i / CPR, c = i - r * CPR;
            uint32_t w4[4] = {stg[j].x, stg[j].y, stg[j].z, stg[j].w};
            if constexpr (U8) {
#pragma unroll
                for (int w = 0; w < 4; w++) w4[w] ^= 0x80808080u;   // x - 128 as int8
                if (c * 16 + 16 > a.dim) {
#pragma unroll
                    for (int w = 0; w < 4; w++) {
                        const int valid = a.dim - (c * 16 + 4 * w);
                        if (valid <= 0) w4[w] = 0u;
                        else if (valid < 4) w4[w] &= (1u << (8 * valid)) - 1u;
                    }
                }
            } else if (c * 4 + 4 > a.dim) {
#pragma unroll
                for (int w = 0; w < 4; w++)
                    if (c * 4 + w >= a.dim) w4[w] = 0u;
            }
            *reinterpret_cast<uint4 *>(buf + (uint32_t)r * (uint32_t)a.lds_pitch + (uint32_t)c * 16u) =
                uint4{w4[0], w4[1], w4[2], w4[3]};
        }
        if (!BOUND && a.b_ids && threadIdx.x < BN)
            reinterpret_cast<uint32_t *>(buf + BN * a.lds_pitch)[BN + threadIdx.x] = side_g;
    };

    // Places the wave's queued candidates: numbers within their rows by LDS
    // counters, one range per row from the row's global counter.
    auto drain = [&]() {
        if (lane < 16) q_cnt[lane] = 0;
        wave_sync();
#pragma unroll 1
        for (int e = lane; e < qn_held; e += WAVE) q_num[e] = (uint8_t)atomicAdd(&q_cnt[q_row[e]], 1);
        wave_sync();
        if (lane < 16) {
            const int n = q_cnt[lane];
            if (n) q_cnt[lane] = atomicAdd(&A.cnt[lrow0 + rw * 16 + lane], n);
        }
        wave_sync();
#pragma unroll 1
        for (int e = lane; e < qn_held; e += WAVE) {
            const int r = q_row[e];
            const int slot = q_cnt[r] + q_num[e];
            if (slot < A.cap) A.cand[(lrow0 + rw * 16 + r) * A.cap + slot] = q_key[e];
        }
        wave_sync();
        qn_held = 0;
    };

    uint32_t best[4] = {~0u, ~0u, ~0u, ~0u};   // bound: smallest distance of the group
    if (t_beg < t_end) {
        fetch_tile(t_beg);
        put_tile(reinterpret_cast<uint8_t *>(smem));
    }
    // the query operands are here: without this the loop's first product waits
    // for every load in flight, the next tile's among them, on each tile
    __builtin_amdgcn_s_waitcnt(0);
    // (filter: a block none of whose rows lets anything pass has nothing to do)
    if (!BOUND && !any_passes) return;
    for (int t = t_beg; t < t_end; t++) {
        uint8_t *const btile = reinterpret_cast<uint8_t *>(smem) + ((t - t_beg) & 1) * buf_bytes;
        uint32_t *const t_norm = reinterpret_cast<uint32_t *>(btile + BN * a.lds_pitch);
        const uint32_t *const t_gid = t_norm + BN;
        __syncthreads();
        if (t + 1 < t_end) fetch_tile(t + 1);
        if (norms) tile_norms<U8, CPR>(btile, a.lds_pitch, nthr, t_norm);   // read after the barrier below

        const uint8_t *bbase = btile + (cw * NCB * 16 + arow) * a.lds_pitch + (U8 ? kg * 16 : kg * KQ * 4);
        i32x4 acc8[NCB];
        f32x4 accf[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; cb++) {
            acc8[cb] = i32x4{0, 0, 0, 0};
            accf[cb] = f32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int c = 0; c < NCH; c++) {
            if constexpr (U8) {
                i32x4 bv[NCB];
#pragma unroll
                for (int cb = 0; cb < NCB; cb++)
                    bv[cb] = *reinterpret_cast<const i32x4 *>(bbase + cb * 16 * a.lds_pitch + c * 64);
#pragma unroll
                for (int cb = 0; cb < NCB; cb++)
                    acc8[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A8[c], bv[cb], acc8[cb], 0, 0, 0);
            } else {
                f32x4 bv[NCB];
#pragma unroll
                for (int cb = 0; cb < NCB; cb++)
                    bv[cb] = *reinterpret_cast<const f32x4 *>(bbase + cb * 16 * a.lds_pitch + c * 16);
#pragma unroll
                for (int j = 0; j < 4; j++)
#pragma unroll
                    for (int cb = 0; cb < NCB; cb++)
                        accf[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(AF[4 * c + j], bv[cb][j],
                                                                          accf[cb], 0, 0, 0);
            }
        }
        if (t + 1 < t_end) put_tile(reinterpret_cast<uint8_t *>(smem) + ((t + 1 - t_beg) & 1) * buf_bytes);
        if (norms) __syncthreads();
        if (!live) continue;
#pragma unroll
        for (int cb = 0; cb < NCB; cb++) {
            const int col = (cw * NCB + cb) * 16 + arow;   // within the tile
            int32_t bn8 = 0;
            float bnf = 0.0f;
            if constexpr (U8) bn8 = (int32_t)t_norm[col];
            else if constexpr (MT == ONNG_L2SQ) bnf = __uint_as_float(t_norm[col]);
            uint32_t dd[4];
            uint64_t hit = 0;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                if constexpr (U8) dd[r] = (uint32_t)(qn8[r] + bn8 - 2 * acc8[cb][r]);
                else if constexpr (MT == ONNG_L2SQ) dd[r] = ord_f32(qnf[r] + bnf - 2.0f * accf[cb][r]);
                else dd[r] = ord_f32(1.0f - accf[cb][r]);
                if (BOUND) best[r] = min(best[r], dd[r]);
                else hit |= ballot(dd[r] < tau[r]);
            }
            if (BOUND || !hit) continue;
            const int64_t c = (int64_t)t * BN + col;
            const bool cok = c < a.nb;
            const uint32_t gid = a.b_ids ? t_gid[col] : (uint32_t)c;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const bool in = cok && rok[r] && dd[r] < tau[r] &&
                                !(a.exclude_self && (int64_t)gid == crow0 + r);
                const uint64_t m = ballot(in);
                if (!m) continue;
                if (qn_held + WAVE > BOUND_QUEUE) drain();
                if (in) {
                    q_key[qn_held + mbcnt(m)] = make_key(dd[r], gid);
                    q_row[qn_held + mbcnt(m)] = (uint8_t)(4 * kg + r);
                }
                qn_held += __popcll(m);
            }
        }
        if (BOUND && (t + 1) % A.group_tiles == 0) {
            const int64_t at = ((int64_t)(t / A.group_tiles) * CW + cw) * 16 + arow;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                if (A.quads) {
                    best[r] = min(best[r], dpp<DPP_QP_1032>(best[r]));
                    best[r] = min(best[r], dpp<DPP_QP_2301>(best[r]));
                }
                if (rok[r] && (!A.quads || (lane & 3) == 0))
                    A.mins[(lcrow0 + r) * A.groups + (A.quads ? at / 4 : at)] = best[r];
                best[r] = ~0u;
            }
        }
    }
    if (!BOUND && qn_held) drain();
}

template <int DT, int MT, int RW, bool BOUND>
const void *topk_bound_fn_nch(int nch) {
    if constexpr (DT == ONNG_U8) {
        switch (nch) {
            case 1: return (const void *)topk_bound_kernel<DT, MT, 1, RW, BOUND>;
            case 2: return (const void *)topk_bound_kernel<DT, MT, 2, RW, BOUND>;
            case 4: return (const void *)topk_bound_kernel<DT, MT, 4, RW, BOUND>;
            default: return (const void *)topk_bound_kernel<DT, MT, 8, RW, BOUND>;
        }
    } else {
        switch (nch) {
            case 2: return (const void *)topk_bound_kernel<DT, MT, 2, RW, BOUND>;
            case 4: return (const void *)topk_bound_kernel<DT, MT, 4, RW, BOUND>;
            case 6: return (const void *)topk_bound_kernel<DT, MT, 6, RW, BOUND>;
            case 7: return (const void *)topk_bound_kernel<DT, MT, 7, RW, BOUND>;
            case 8: return (const void *)topk_bound_kernel<DT, MT, 8, RW, BOUND>;
            case 12: return (const void *)topk_bound_kernel<DT, MT, 12, RW, BOUND>;
            default: return (const void *)topk_bound_kernel<DT, MT, 16, RW, BOUND>;
        }
    }
}

// the kernel for rw = 1, 4 or 8 row waves, bound or filter
template <int DT, int MT>
const void *topk_bound_fn(int nch, int rw, bool bound) {
    switch (rw) {
        case 1: return bound ? topk_bound_fn_nch<DT, MT, 1, true>(nch) : topk_bound_fn_nch<DT, MT, 1, false>(nch);
        case 4: return bound ? topk_bound_fn_nch<DT, MT, 4, true>(nch) : topk_bound_fn_nch<DT, MT, 4, false>(nch);
        default: return bound ? topk_bound_fn_nch<DT, MT, 8, true>(nch) : topk_bound_fn_nch<DT, MT, 8, false>(nch);
    }
}

const void *topk_bound_fn_u8(int nch, int rw, bool bound);
const void *topk_bound_fn_l2(int nch, int rw, bool bound);
const void *topk_bound_fn_cosine(int nch, int rw, bool bound);

}  // namespace topk_detail
}  // namespace onng
