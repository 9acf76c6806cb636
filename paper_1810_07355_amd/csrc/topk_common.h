// Shared by the two top-k kernels (topk.hip, topk_wide.hip): the kernel
// argument block, tile geometry and the int8 operand staging.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "onng_internal.h"
#include "wave.h"

namespace onng {
namespace topk_detail {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BN = 64;        // base rows per tile
// Per-row list capacity (k rounded up to 8 keys) and candidate slots: a
// tile adds at most BN candidates to a row, whose buffer is merged once it
// holds more than cb - BN.  Small k takes 80 slots (merges after 16
// candidates), which halves the buffer's LDS.
__host__ __device__ inline int topk_kcap(int k) { return (k + 7) / 8 * 8; }
__host__ __device__ inline int topk_cb(int k) { return k <= 16 ? 80 : 128; }

// A staged row is NCH * 64 bytes: u8, NCH k-steps of 64 components (a lane
// feeds 16 of them per step); f32, 4 k-groups of KQ = 4 * NCH components,
// k-group kg covering [kg * KQ, kg * KQ + KQ), so that a lane reads four
// k-steps of its B column with one 16-byte LDS read.  NCH is a compile-time
// constant of the kernel, taken from a short list (rows are zero-extended up
// to it), so the contraction unrolls into one straight run of LDS reads and
// MFMAs.
__host__ __device__ inline int nch_for(int dtype, int dim) {
    if (dtype == ONNG_U8) {
        const int need = (dim + 63) / 64;
        return need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 8;
    }
    const int need = (dim + 15) / 16;
    return need <= 2 ? 2 : need <= 4 ? 4 : need <= 6 ? 6 : need <= 7 ? 7 : need <= 8 ? 8
           : need <= 12 ? 12 : 16;
}

struct TopkArgs {
    const uint8_t *q;
    int64_t q_pitch;
    int64_t nq;
    const uint8_t *b;         // base rows (or gathered candidate rows)
    int64_t b_pitch;
    int64_t nb;
    const int32_t *b_ids;     // global id of each base row (null: the row index)
    const void *qn;           // query norms (int32 or float), null for cosine
    const void *bn;           // base norms
    int32_t dim;
    int32_t k;
    int32_t kcap;             // list capacity per row (topk_kcap)
    int32_t cb;               // candidate slots per row (topk_cb)
    int32_t bm;               // query rows per block (16 per wave)
    int32_t exclude_self;
    int32_t rotate;           // rows and candidates are the same rows: start at the own tile
    int32_t lds_pitch;        // bytes per staged base row
    int32_t *out_ids;
    void *out_d;
    int32_t side_norms;       // stage the tile's base norms in LDS (L2 metrics)
    int32_t splits;           // blocks sharing one row block's base tiles
    int32_t tiles_per_split;
    uint64_t *part;           // splits > 1: [nq][splits][k] keys of each part
    const int32_t *only;      // null, or [1 + nq]: only[0] != 0 when any row is to be
                              // done, only[1 + row] != 0 when this one is
};

// 16 int8 values of (x - 128) at row bytes [c, c+16), zero past dim
__device__ __forceinline__ i32x4 shifted16(const uint8_t *row, int c, int dim) {
    i32x4 out;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            int idx = c + 4 * w + b;
            uint32_t byte = idx < dim ? (uint32_t)(uint8_t)((int)row[idx] - 128) : 0u;
            v |= byte << (8 * b);
        }
        out[w] = (int32_t)v;
    }
    return out;
}

constexpr uint32_t SAMPLE_ODD = 0x9E3779B1u;

// base row of sampled column i: odd multiples modulo a power of two visit
// every sample once, neighbouring columns far apart (rows in locality order
// would put a query's near rows into one group, whose minimum counts once)
__device__ __forceinline__ int64_t sample_row(uint32_t i, int ns_log2, int64_t nb) {
    const uint32_t j = (i * SAMPLE_ODD) & ((1u << ns_log2) - 1u);
    return (int64_t)(((uint64_t)j * (uint64_t)nb) >> ns_log2);
}

// Norms of a staged tile's BN rows (CPR 16-byte chunks each) by nthr threads,
// sixteen lanes per row: int32 of the shifted u8 rows; f32 in the order of
// norms_kernel<float> (one component per lane, chains 64 apart, then lanes 32, 16,
// .. 1 apart), four of its lanes in each of these, so the same bits.
template <bool U8, int CPR>
__device__ __forceinline__ void tile_norms(const uint8_t *tile, int lds_pitch, int nthr, uint32_t *out) {
    const int l = threadIdx.x & 15;
    for (int r = threadIdx.x / 16; r < BN; r += nthr / 16) {
        const uint8_t *row = tile + (uint32_t)r * (uint32_t)lds_pitch;
        if constexpr (U8) {
            int32_t s = 0;
            for (int c = l; c < CPR; c += 16) {
                const i32x4 x = *reinterpret_cast<const i32x4 *>(row + c * 16);
#pragma unroll
                for (int w = 0; w < 4; w++) s = __builtin_amdgcn_sdot4(x[w], x[w], s, false);
            }
            s = group_sum<16>(s);
            if (l == 0) out[r] = (uint32_t)s;
        } else {
            float p[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int c = l; c < CPR; c += 16) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(row + c * 16);
#pragma unroll
                for (int e = 0; e < 4; e++) p[e] = fmaf(x[e], x[e], p[e]);
            }
#pragma unroll
            for (int e = 0; e < 4; e++) p[e] = group_sum<16>(p[e]);
            const float s = (p[0] + p[2]) + (p[1] + p[3]);
            if (l == 0) out[r] = __float_as_uint(s);
        }
    }
}

// Bytes of a staged row: what the MFMA operands read (u8: whole 64-byte
// k-steps; f32: 4 k-groups of KQ components), rounded up to an odd number of
// 16-byte chunks, which spreads the 16 rows read together over the LDS banks
// (no more than two rows per bank group).
inline int lds_pitch_for(int dtype, int32_t dim) {
    int p = nch_for(dtype, dim) * 64;
    if ((p / 16) % 2 == 0) p += 16;
    return p;
}

// ---- u8 rows of at most 128 components, many query rows ------------------
// The kernel above keeps every row's list and candidate buffer in LDS: for
// k = 100 that is one block of 64 rows per compute unit, one wave per SIMD,
// whose staging, barriers and epilogue never overlap its MFMAs.  Here a wave
// owns WIDE_RB * 16 = 64 query rows, whose A operands stay in registers for
// the whole sweep, and the lists and candidate buffers live in global memory.
// After the first tiles a row's threshold is tight and few values pass it,
// so those buffers are rarely touched; the LDS holds the staged tile, the
// per-row thresholds and counters and one merge list per wave, so several
// blocks share a compute unit and one wave's epilogue overlaps another's
// MFMAs.  The epilogue's common case is one comparison per distance (the
// column's norm enters as the MFMA chain's initial accumulator, below).
constexpr int WIDE_RB = 4;       // 16-row blocks per wave
constexpr int WIDE_ROWS = 4 * WIDE_RB * 16;   // query rows per block (4 waves)
// Base rows per staged tile: 128 (one barrier pair per 32 MFMAs of each
// 16-row block; 64 was measured 7% slower on the 1M build).
constexpr int WBN = 128;
constexpr int WIDE_CB = 2 * WBN; // global candidate slots per row (a tile adds at most WBN)

__host__ __device__ inline size_t wide_lds_bytes(int lds_pitch, int kcap) {
    return (size_t)WBN * lds_pitch + (size_t)WBN * 12 + (size_t)WIDE_ROWS * 20 +
           (size_t)4 * (kcap + WAVE) * 8;
}

onng_status launch_topk_wide(const TopkArgs &a, int nch, uint64_t *glist, uint64_t *gcand,
                             hipStream_t st);

// f32 rows of at most 128 components: the bf16-screened wide kernel.
constexpr int FW_RB = 2;                  // 16-row blocks per wave
constexpr int FW_ROWS = 4 * FW_RB * 16;   // query rows per block (4 waves)
constexpr int FW_NCH = 4;                 // 64-byte k-steps: 128 bf16 components
constexpr int FW_BN = 64;                 // base rows per staged tile
constexpr int FW_CB = 2 * FW_BN;          // global candidate slots per row
constexpr int FW_LDS_PITCH = FW_NCH * 64 + 16;   // odd count of 16-byte chunks
// |dot(bf16(x), bf16(y)) in f32 - dot(x, y)| <= FW_C |x| |y| for at most 128
// components: 2^-7 + 2^-16 for the rounded factors, 128 * 2^-24 for the sum.
constexpr float FW_C = 0.0078278f + 1.6e-5f;

struct FwRows {
    const uint8_t *q;       // bf16 query rows
    int64_t q_pitch;
    const uint8_t *b;       // bf16 base rows
    int64_t b_pitch;
    const float *ymax;      // max |y| over the base rows
};

__host__ __device__ inline size_t fw_lds_bytes(int kcap) {
    return (size_t)FW_BN * FW_LDS_PITCH + (size_t)FW_BN * 4 + (size_t)FW_ROWS * 20 +
           (size_t)4 * (kcap + WAVE + 64) * 8;
}

onng_status launch_topk_wide_f32(const TopkArgs &a, const onng_vectors *Q, bool same_rows,
                                 uint8_t *qh, uint8_t *bh, uint32_t *ymax, uint64_t *glist,
                                 uint32_t *gcand, hipStream_t st);

// ---- many query rows by a bound and a filter (topk_wide_bound.hip) -------
// The two passes of topk_bound.h for many query rows: a wave holds 64 of them
// (four 16-row blocks), whose operands stay in registers for the sweep, so each
// operand read from LDS feeds four matrix instructions.
constexpr int WB_ROWS = 256;              // query rows per block of four waves
constexpr int WB_QUEUE = 256;             // candidates a wave holds before it places them
constexpr int64_t WB_CHUNK = 32768;       // query rows whose candidates are held at a time

struct WidePlan {
    bool use = false;
    int nch = 0;                          // 64-byte k-steps per row
    int64_t chunk = 0;                    // query rows per launch, at most WB_CHUNK
    int ns_log2 = 0, group_tiles = 0, groups = 0, cap = 0;
    int splits[2] = {1, 1}, per_split[2] = {0, 0};   // bound, filter
};
// workspace of the wide passes, carved by the caller
struct WideBufs {
    uint32_t *mins;      // [chunk][groups]
    uint32_t *tau;       // [chunk]
    int32_t *cnt;        // [chunk]
    uint64_t *cand;      // [chunk][cap]
    int32_t *redo;       // [1 + nq]: rows left to the older kernel
    uint8_t *bh, *qh;    // converted rows (int8, or f16 of f32 data)
    float *side;         // [nb] (f32)
    float *len;          // [2]: largest |y| of the base, of the queries (f32)
};
WidePlan wide_bound_plan(const onng_vectors *Q, int64_t nb, int32_t k);
onng_status launch_wide_bound(const TopkArgs &a, const onng_vectors *Q, bool same_rows, const WidePlan &P,
                              const WideBufs &w, hipStream_t st);

// Per row an upper bound of the rank-th smallest of its group minima plus `past`,
// its counter cleared (and *clear, when given), or, where more than `most` minima
// are within the bound, `none` and the counter past cap; its candidates sorted and
// the k first (drop_own: without the row's own id) written at row0 + row, or redo[1 + row0 + row] and redo[0] set
// (topk.hip).
void launch_bound_select(const uint32_t *mins, int64_t nq, int groups, int rank, int most, int top, int low,
                         int cap, uint32_t past, uint32_t none, uint32_t *tau, int32_t *cnt, int32_t *clear, hipStream_t st);
// minima that stand for cap base rows
inline int bound_most(int cap, int ns_log2, int64_t nb) { return (int)(((int64_t)cap << ns_log2) / nb); }
void launch_bound_sort(bool u8, const uint64_t *cand, int cap, const int32_t *cnt, int64_t nq, int k,
                       bool drop_own, int32_t *ids, void *dists, int32_t *redo, int64_t row0, hipStream_t st);

}  // namespace topk_detail
}  // namespace onng
