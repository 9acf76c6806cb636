// Exact top-k for many query rows by a bound and a filter (topk_bound.h says how
// the two passes work).  A wave holds 64 query rows.
//
// u8 rows: int8 products, exact.  f32 rows (at most 128 components): the passes
// run on f16 copies of the rows, scaled by a power of two, whose dot products
// are within a bound of the exact ones; the bound widens both passes, so every
// row that belongs to the result is among the candidates.  (bf16, with the same
// rate, would widen them eight times as much.)  Per row the
// candidates are then narrowed once more by their own k-th best approximate
// value, and the survivors' distances computed in f32 from the f32 rows (one
// chain in component order, as topk_f32_wide_kernel computes them): the result
// is the f32 brute force's.
//
// Bound by instruction issue: the matrix cores and the vector ALU (compares,
// maxima, candidates) each take about 30% of the cycles.  kNN of 100,003 x 100
// f32, cosine, k 100: 24.6 -> 5.7 ms against the kernel that keeps lists (rows in
// locality order); 70,000 x 128 u8, k 100: 14.0 -> 2.5; 1M x 100 f32: 506 -> 387.
// Rows that are left to that kernel cost its whole sweep besides: 3000 equal rows
// among the 70,000 14.0 -> 15.2 ms, among 100,003 f32 rows (in no order) 46.3 -> 35.9;
// 70,000 rows of 100 distinct ones 10.2 -> 13.1.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "onng_internal.h"
#include "topk_common.h"
#include "wave.h"

namespace onng {
namespace topk_detail {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

struct WideArgs {
    TopkArgs t;              // q, b: the converted rows, pitch NCH * 64 bytes
    const uint32_t *side;    // per base row: u8 |y'|^2, f32 L2 -|y|^2 / 2 scaled
    int64_t row0;            // first query row of this chunk
    int32_t rows;            // query rows in the chunk
    int32_t ns_log2, group_tiles, groups;
    uint32_t *mins;
    const uint32_t *tau;
    int32_t *cnt;
    uint64_t *cand;
    int32_t cap;
    const float *len;        // f32: largest |y| of the base, of the queries
    int32_t drop_own;        // f32: the row's own id is left out at the end
};

// ---- f32 rows as f16 ------------------------------------------------------
// Scale: the power of two that takes the longest row to at most 2^8, so that
// components and products are far from f16's and f32's limits.  A squared length
// past f32's range leaves no such power: other rows may then overflow f16, whose
// products say nothing, and every row is left to the list kernel.
__device__ __forceinline__ bool wide_has_scale(const float *len) { return fmaxf(len[0], len[1]) < 1e30f; }

__device__ __forceinline__ float wide_scale(const float *len) {
    const float m = fmaxf(len[0], len[1]);
    if (!(m > 0.0f) || !wide_has_scale(len)) return 1.0f;
    int e;
    frexpf(m, &e);   // m <= 2^e
    return ldexpf(1.0f, min(max(8 - e, -90), 90));
}

// |f16 dot in f32 - exact dot| of scaled rows of lengths X, Y, at most 128
// components: each factor rounded to 11 significant bits (2^-11 relative, twice)
// or, below 2^-14, off by at most 2^-14 (absolute; sqrt(128) of them against the
// other row's length); 128 f32 additions.  The slack covers the f32 rounding of
// norms, thresholds and recomputed distances (at most 128 additions of 2^-24).
__device__ __forceinline__ float wide_margin(float X, float Y, float s, bool cosine) {
    const float dot = (0x1.02p-10f + 512.0f * 0x1p-24f) * X * Y + 11.4f * 0x1p-14f * (X + Y) + 128.0f * 0x1p-28f;
    return dot + 3e-5f * (X * X + Y * Y + (cosine ? s * s : 0.0f));
}

__global__ void len_zero_kernel(float *len) { len[threadIdx.x] = 0.0f; }

// len = max(len, max_i sqrt(n2[i])) (non-negative floats order as their bits)
__global__ void len_max_kernel(const float *n2, int64_t n, float *len) {
    float m = 0.0f;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        m = fmaxf(m, n2[i]);
    for (int s = 32; s >= 1; s >>= 1) m = fmaxf(m, __shfl_xor(m, s));
    if (lane_id() == 0 && m > 0.0f) atomicMax(reinterpret_cast<unsigned int *>(len), __float_as_uint(sqrtf(m)));
}

// Converted rows of NCH * 64 bytes, 16 bytes per thread, zero past dim: f16 of
// the scaled components, or u8 components as int8 (x - 128).
__global__ void to_f16_kernel(const uint8_t *src, int64_t pitch, int64_t n, int dim, const float *len,
                              uint8_t *dst, int dst_pitch) {
    const int per = dst_pitch / 16;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * per) return;
    const float s = wide_scale(len);
    const int64_t r = i / per;
    const int c = (int)(i - r * per) * 8;
    const float *x = reinterpret_cast<const float *>(src + r * pitch);
    f16x8 o;
#pragma unroll
    for (int e = 0; e < 8; e++) o[e] = c + e < dim ? (_Float16)(x[c + e] * s) : (_Float16)0.0f;
    *reinterpret_cast<f16x8 *>(dst + r * dst_pitch + (int64_t)c * 2) = o;
}

__global__ void to_i8_kernel(const uint8_t *src, int64_t pitch, int64_t n, int dim, uint8_t *dst, int dst_pitch) {
    const int per = dst_pitch / 16;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * per) return;
    const int64_t r = i / per;
    const int c = (int)(i - r * per) * 16;
    *reinterpret_cast<i32x4 *>(dst + r * dst_pitch + c) = shifted16(src + r * pitch, c, dim);
}

// start value of a column's products (f32, squared L2)
__global__ void side_f32_kernel(const float *n2, int64_t n, const float *len, float *side) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float s = wide_scale(len);
    side[i] = -0.5f * n2[i] * s * s;
}

// ---- the passes -----------------------------------------------------------
// D of a pair: u8 <x', y'> - floor(|y'|^2 / 2) (the chain starts from the
// column's -floor(|y'|^2 / 2)); f32 <x, y> - |y|^2 / 2 (squared L2) or <x, y>
// (cosine), scaled.  Larger is nearer.
template <int DT, int MT, int NCH, bool BOUND>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) topk_wide_bound_kernel(WideArgs A) {
    constexpr bool U8 = DT == ONNG_U8;
    typedef typename std::conditional<U8, i32x4, f16x8>::type op_t;
    typedef typename std::conditional<U8, i32x4, f32x4>::type acc_t;
    typedef typename std::conditional<U8, int32_t, float>::type val_t;
    constexpr int RB = WB_ROWS / 4 / 16;
    constexpr int CPR = NCH * 4;              // 16-byte chunks of a staged row
    constexpr bool side = U8 || MT == ONNG_L2SQ;
    const TopkArgs &a = A.t;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int wv = uni(threadIdx.x / WAVE);
    const int lrow0 = blockIdx.x * WB_ROWS + wv * WAVE;   // the wave's first row within the chunk
    const int arow = lane & 15, kg = lane >> 4;

    // LDS: two of [tile BN * NCH * 64][side BN], filter: per wave [queue keys]
    // [counts 64][queue rows][numbers].  A tile row's 16-byte pieces sit at
    // their place xor the row's low bits, so that the 16 rows read together
    // spread over all banks; the copies from global memory go straight to LDS
    // (64 consecutive pieces per wave and instruction) and need no registers.
    constexpr uint32_t buf_bytes = BN * (NCH * 64 + 4);
    constexpr int SWZ = CPR - 1;   // (CPR = 12: rows' low two bits, below)
    char *wq = smem + 2 * buf_bytes + (size_t)wv * (WB_QUEUE * 10 + 256);
    uint64_t *q_key = reinterpret_cast<uint64_t *>(wq);
    int32_t *q_cnt = reinterpret_cast<int32_t *>(q_key + WB_QUEUE);
    uint8_t *q_row = reinterpret_cast<uint8_t *>(q_cnt + WAVE);
    uint8_t *q_num = q_row + WB_QUEUE;
    int held = 0;

    op_t X[RB][NCH];
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
        const int lr = lrow0 + rb * 16 + arow;
        const bool ok = lr < A.rows;
        const uint8_t *qp = a.q + (A.row0 + (ok ? lr : 0)) * a.q_pitch;
#pragma unroll
        for (int s = 0; s < NCH; s++)
            X[rb][s] = ok ? *reinterpret_cast<const op_t *>(qp + s * 64 + kg * 16) : op_t{};
    }
    float scale = 1.0f;
    if constexpr (!U8) scale = wide_scale(A.len);
    // filter: the smallest D that passes, per row this lane sees in C (row
    // rb*16 + 4*kg + r).  u8: d = |x'|^2 + (bn & 1) - 2D, and the bound's D gives
    // d <= |x'|^2 + 1 - 2D; one more unit of slack in D, the exact test follows.
    val_t lim[RB][4], best[RB][4];
    auto each_row = [&](auto f) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int r = 0; r < 4; r++) f(rb, r, lrow0 + rb * 16 + 4 * kg + r);
    };
    each_row([&](int rb, int r, int lr) {
        if constexpr (BOUND) {
            best[rb][r] = U8 ? (val_t)INT32_MIN : (val_t)-__builtin_inff();
        } else if constexpr (U8) {
            const uint32_t t = lr < A.rows ? ~A.tau[lr] ^ 0x80000000u : 0x7FFFFFFFu;
            lim[rb][r] = lr < A.rows ? (int32_t)t - 1 : INT32_MAX;
        } else {
            float th = __builtin_inff();
            if (lr < A.rows) {
                const float x = sqrtf(reinterpret_cast<const float *>(a.qn)[A.row0 + lr]) * scale;
                const float m = wide_margin(x, A.len[0] * scale, scale, MT == ONNG_COSINE);
                th = unord_f32(~A.tau[lr]) - 2.0f * m;
                if (th != th) th = -__builtin_inff();   // (no bound: all pass, the row is redone)
            }
            lim[rb][r] = th;
        }
    });
    const bool live = lrow0 < A.rows;

    const int ntiles = BOUND ? (1 << A.ns_log2) / BN : (int)((a.nb + BN - 1) / BN);
    const int t_beg = blockIdx.y * a.tiles_per_split;
    const int t_end = min(ntiles, t_beg + a.tiles_per_split);
    // piece c of tile row r sits at place swz(r, c) of the row
    auto swz = [](int r, int c) { return NCH == 3 ? c ^ (r & 3) : c ^ (r & SWZ); };
    auto tile_row = [&](int t, int r) {
        const int64_t i = (int64_t)t * BN + r;
        if (BOUND) return sample_row((uint32_t)i, A.ns_log2, a.nb);
        return i < a.nb ? i : a.nb - 1;   // (rows past the end repeat the last; never taken)
    };
    auto fetch_tile = [&](int t, char *buf) {
#pragma unroll
        for (int j = 0; j < CPR / 4; j++) {
            const int base = (wv * (CPR / 4) + j) * WAVE;   // the wave's first piece
            const int i = base + lane;
            const int r = i / CPR, c = swz(r, i % CPR);
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(a.b + tile_row(t, r) * (NCH * 64) + c * 16),
                (__attribute__((address_space(3))) void *)(buf + base * 16), 16, 0, 0);
        }
        if (side && wv == 0)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(A.side + tile_row(t, lane)),
                (__attribute__((address_space(3))) void *)(buf + BN * NCH * 64), 4, 0, 0);
    };
    // Queue entry: the bits of D, and the column (u8: with |y'|^2's low bit on
    // top).  Places the wave's queued candidates: numbers within their rows by
    // LDS counters, one range per row from the row's global counter.
    constexpr uint8_t Q_SELF = 255;   // the row itself, left out
    auto drain = [&]() {
        q_cnt[lane] = 0;
        wave_sync();
#pragma unroll 1
        for (int e = lane; e < held; e += WAVE) {
            const int r = q_row[e];
            if (a.exclude_self && (int64_t)((uint32_t)q_key[e] & 0x7FFFFFFFu) == A.row0 + lrow0 + r) q_row[e] = Q_SELF;
            else q_num[e] = (uint8_t)atomicAdd(&q_cnt[r], 1);
        }
        wave_sync();
        const int n = q_cnt[lane];
        if (n) q_cnt[lane] = atomicAdd(&A.cnt[lrow0 + lane], n);
        wave_sync();
#pragma unroll 1
        for (int e = lane; e < held; e += WAVE) {
            const int r = q_row[e];
            if (r == Q_SELF) continue;
            const int slot = q_cnt[r] + q_num[e];
            const uint32_t hi = (uint32_t)(q_key[e] >> 32), lo = (uint32_t)q_key[e];
            const uint32_t col = lo & 0x7FFFFFFFu;
            uint64_t key;
            if constexpr (U8) {   // d = |x'|^2 + (|y'|^2 & 1) - 2D
                const int32_t qn = reinterpret_cast<const int32_t *>(a.qn)[A.row0 + lrow0 + r];
                key = make_key((uint32_t)(qn + (int32_t)(lo >> 31) - 2 * (int32_t)hi),
                               a.b_ids ? (uint32_t)a.b_ids[col] : col);
            } else {
                key = make_key(~ord_f32(__uint_as_float(hi)), col);
            }
            if (slot < A.cap) A.cand[(int64_t)(lrow0 + r) * A.cap + slot] = key;
        }
        wave_sync();
        held = 0;
    };

    if (t_beg < t_end) fetch_tile(t_beg, smem);
    for (int t = t_beg; t < t_end; t++) {
        char *const btile = smem + ((t - t_beg) & 1) * buf_bytes;
        const uint32_t *const sd = reinterpret_cast<const uint32_t *>(btile + BN * NCH * 64);
        __builtin_amdgcn_s_waitcnt(0);   // this wave's copies of the tile (and the operands) are here
        __syncthreads();
        if (t + 1 < t_end) fetch_tile(t + 1, smem + ((t + 1 - t_beg) & 1) * buf_bytes);
        if (live) {
#pragma unroll 1
            for (int cb = 0; cb < BN / 16; cb++) {
                const int col = cb * 16 + arow;
                const char *bp = btile + (uint32_t)col * (NCH * 64);
                op_t Y[NCH];
#pragma unroll
                for (int s = 0; s < NCH; s++) Y[s] = *reinterpret_cast<const op_t *>(bp + swz(col, s * 4 + kg) * 16);
                val_t c0 = 0;
                if constexpr (U8) c0 = -((int32_t)sd[col] >> 1);
                else if constexpr (MT == ONNG_L2SQ) c0 = __uint_as_float(sd[col]);
                const acc_t start = acc_t{c0, c0, c0, c0};
                acc_t acc[RB];
#pragma unroll
                for (int s = 0; s < NCH; s++)
#pragma unroll
                    for (int rb = 0; rb < RB; rb++) {
                        if constexpr (U8)
                            acc[rb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(X[rb][s], Y[s], s ? acc[rb] : start, 0, 0, 0);
                        else
                            acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(X[rb][s], Y[s], s ? acc[rb] : start, 0, 0, 0);
                    }
                if constexpr (BOUND) {
                    each_row([&](int rb, int r, int) { best[rb][r] = max(best[rb][r], acc[rb][r]); });
                } else {
                    uint64_t hit = 0;
                    each_row([&](int rb, int r, int) { hit |= ballot(acc[rb][r] >= lim[rb][r]); });
                    if (!hit) continue;
                    const uint32_t c = (uint32_t)t * BN + col;
                    const uint64_t okm = ballot((int64_t)c < a.nb);
                    uint32_t lo = c;
                    if constexpr (U8) lo |= sd[col] << 31;
                    const uint32_t row4 = 4 * kg;
                    each_row([&](int rb, int r, int) {
                        const uint64_t m = ballot(acc[rb][r] >= lim[rb][r]) & okm;
                        if (!m) return;
                        if (held + WAVE > WB_QUEUE) drain();
                        if ((m >> lane) & 1) {
                            const int at = held + mbcnt(m);
                            const val_t v = acc[rb][r];
                            q_key[at] = make_key(__builtin_bit_cast(uint32_t, v), lo);
                            q_row[at] = (uint8_t)(row4 + (rb * 16 + r));
                        }
                        held += __popcll(m);
                    });
                }
            }
        }
        if constexpr (BOUND) {
            if ((t + 1) % A.group_tiles == 0) {
                const int64_t at = (int64_t)(t / A.group_tiles) * 16 + arow;
                each_row([&](int rb, int r, int lr) {
                    uint32_t o;
                    if constexpr (U8) o = ~((uint32_t)best[rb][r] ^ 0x80000000u);
                    else o = ~ord_f32(best[rb][r]);
                    if (lr < A.rows) A.mins[(int64_t)lr * A.groups + at] = o;
                    best[rb][r] = U8 ? (val_t)INT32_MIN : (val_t)-__builtin_inff();
                });
            }
        }
    }
    if (!BOUND && held) drain();
}

// ---- f32: from a row's candidates to its k nearest ------------------------
// One wave per row.  The k-th best approximate value of the candidates (found
// by its bits, VPL candidates per lane) less twice the margin drops the ones
// that cannot belong to the result; the survivors' rows are staged through LDS
// 32 components at a time (a row's 128 bytes by eight lanes) and every lane
// computes one distance; a bitonic network orders them.
constexpr int FIN_PITCH = 144;   // bytes of a staged piece: an odd number of 16-byte chunks

template <int MT, int VPL>
__global__ void __launch_bounds__(64) wide_finish_kernel(WideArgs A, const uint8_t *q, int64_t q_pitch,
                                                         const uint8_t *b, int64_t b_pitch, int32_t *redo) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint64_t *keys = reinterpret_cast<uint64_t *>(smem);              // [cap]
    char *stage = smem + (size_t)A.cap * 8;                           // [64][FIN_PITCH]
    float *qs = reinterpret_cast<float *>(stage + WAVE * FIN_PITCH);  // [128]
    const TopkArgs &a = A.t;
    const int lane = lane_id();
    const int lr = blockIdx.x;
    const int64_t row = A.row0 + lr;
    const int n = uni(A.cnt[lr]);
    const int64_t avail = a.nb - (a.exclude_self || A.drop_own ? 1 : 0);
    const int need = (int)min<int64_t>(a.k, avail);
    bool bad = n > A.cap || n < need || !wide_has_scale(A.len);
    const uint64_t *src = A.cand + (int64_t)lr * A.cap;
    uint64_t key[VPL];
    if (!bad) {
#pragma unroll
        for (int i = 0; i < VPL; i++) key[i] = i * WAVE + lane < n ? src[i * WAVE + lane] : KEY_MAX;
        if (A.drop_own) {
            int own = 0;
#pragma unroll
            for (int i = 0; i < VPL; i++) {
                const bool is = i * WAVE + lane < n && (int64_t)a.b_ids[(uint32_t)key[i]] == row;
                if (is) key[i] = KEY_MAX;
                own += __popcll(ballot(is));
            }
            bad = n - own < need;
        }
    }
    if (lane == 0) {
        redo[1 + row] = bad;
        if (bad) redo[0] = 1;
    }
    if (bad) return;
    const float *qf = reinterpret_cast<const float *>(q + row * q_pitch);
    for (int c = lane; c < 128; c += WAVE) qs[c] = c < a.dim ? qf[c] : 0.0f;
    // the k-th smallest of ~ord(D)
    uint32_t v = 0;
    for (int bit = 31; bit >= 8; bit--) {
        const uint32_t trial = v | ((1u << bit) - 1u);
        int c = 0;
#pragma unroll
        for (int i = 0; i < VPL; i++) c += __popcll(ballot((uint32_t)(key[i] >> 32) <= trial));
        if (c < a.k) v |= 1u << bit;
    }
    v |= 0xFFu;
    const float scale = wide_scale(A.len);
    const float x = sqrtf(reinterpret_cast<const float *>(a.qn)[row]) * scale;
    const float m = wide_margin(x, A.len[0] * scale, scale, MT == ONNG_COSINE);
    const float dmin = unord_f32(~v) - 2.0f * m;
    int ns = 0;
#pragma unroll
    for (int i = 0; i < VPL; i++) {
        const bool in = key[i] != KEY_MAX && !(unord_f32(~(uint32_t)(key[i] >> 32)) < dmin);
        const uint64_t bal = ballot(in);
        if (in) keys[ns + mbcnt(bal)] = key[i];
        ns += __popcll(bal);
    }
    wave_sync();
    for (int s0 = 0; s0 < ns; s0 += WAVE) {
        const int mine = s0 + lane;
        float acc = 0.0f;
        for (int c0 = 0; c0 < a.dim; c0 += 32) {
            // eight lanes per row, eight rows per step
            float4 g[8];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int r = s0 + j * 8 + lane / 8;
                const int c = c0 + (lane & 7) * 4;
                g[j] = float4{0.0f, 0.0f, 0.0f, 0.0f};
                if (r < ns && c < a.dim)
                    g[j] = *reinterpret_cast<const float4 *>(b + (int64_t)(uint32_t)keys[r] * b_pitch + (int64_t)c * 4);
                if (c + 1 >= a.dim) g[j].y = 0.0f;
                if (c + 2 >= a.dim) g[j].z = 0.0f;
                if (c + 3 >= a.dim) g[j].w = 0.0f;
            }
            wave_sync();
#pragma unroll
            for (int j = 0; j < 8; j++)
                *reinterpret_cast<float4 *>(stage + (j * 8 + lane / 8) * FIN_PITCH + (lane & 7) * 16) = g[j];
            wave_sync();
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const float4 y4 = *reinterpret_cast<const float4 *>(stage + lane * FIN_PITCH + u * 16);
                const float4 x4 = *reinterpret_cast<const float4 *>(qs + c0 + u * 4);
                if constexpr (MT == ONNG_COSINE) {
                    acc = fmaf(x4.x, y4.x, acc);
                    acc = fmaf(x4.y, y4.y, acc);
                    acc = fmaf(x4.z, y4.z, acc);
                    acc = fmaf(x4.w, y4.w, acc);
                } else {
                    const float d0 = x4.x - y4.x, d1 = x4.y - y4.y, d2 = x4.z - y4.z, d3 = x4.w - y4.w;
                    acc = fmaf(d0, d0, acc);
                    acc = fmaf(d1, d1, acc);
                    acc = fmaf(d2, d2, acc);
                    acc = fmaf(d3, d3, acc);
                }
            }
        }
        wave_sync();
        if (mine < ns) {
            const uint32_t col = (uint32_t)keys[mine];
            const float d = MT == ONNG_COSINE ? 1.0f - acc : acc;
            keys[mine] = make_key(ord_f32(d), a.b_ids ? (uint32_t)a.b_ids[col] : col);
        }
    }
    wave_sync();
    auto put = [&](int i, uint64_t k) {
        a.out_ids[row * a.k + i] = i < ns ? (int32_t)(uint32_t)k : -1;
        reinterpret_cast<float *>(a.out_d)[row * a.k + i] = i < ns ? unord_f32((uint32_t)(k >> 32)) : __builtin_inff();
    };
    if (ns <= WAVE) {
        uint64_t k = lane < ns ? keys[lane] : KEY_MAX;
        k = wave_sort(k, pow2_at_least(max(ns, 1)));
        if (lane < a.k) put(lane, k);
        for (int i = WAVE + lane; i < a.k; i += WAVE) put(i, KEY_MAX);
        return;
    }
    const int w = pow2_at_least(ns);
    for (int i = ns + lane; i < w; i += WAVE) keys[i] = KEY_MAX;
    for (int size = 2; size <= w; size <<= 1)
        for (int d = size >> 1; d > 0; d >>= 1) {
            wave_sync();
            for (int t = lane; t < w / 2; t += WAVE) {
                const int i = 2 * t - (t & (d - 1));   // lower of the pair (i, i + d)
                const uint64_t lo = keys[i], hi = keys[i + d];
                if ((lo > hi) == ((i & size) == 0)) keys[i] = hi, keys[i + d] = lo;
            }
        }
    wave_sync();
    for (int i = lane; i < a.k; i += WAVE) put(i, i < w ? keys[i] : KEY_MAX);
}

template <int DT, int MT, bool BOUND>
const void *wide_fn(int nch) {
    switch (nch) {
        case 1: return (const void *)topk_wide_bound_kernel<DT, MT, 1, BOUND>;
        case 2: return (const void *)topk_wide_bound_kernel<DT, MT, 2, BOUND>;
        case 3: if constexpr (DT == ONNG_F32) return (const void *)topk_wide_bound_kernel<DT, MT, 3, BOUND>;
        default: if constexpr (DT == ONNG_F32) return (const void *)topk_wide_bound_kernel<DT, MT, 4, BOUND>;
    }
    return nullptr;
}

size_t wide_lds(int pitch, bool filter) {
    return (size_t)2 * BN * (pitch + 4) + (filter ? (size_t)4 * (WB_QUEUE * 10 + 256) : 0);
}

template <int MT>
const void *finish_fn(int cap) {
    return cap <= 256    ? (const void *)wide_finish_kernel<MT, 4>
           : cap <= 512  ? (const void *)wide_finish_kernel<MT, 8>
           : cap <= 1024 ? (const void *)wide_finish_kernel<MT, 16>
                         : (const void *)wide_finish_kernel<MT, 32>;
}

}  // namespace

WidePlan wide_bound_plan(const onng_vectors *Q, int64_t nb, int32_t k) {
    WidePlan P;
    const bool u8 = Q->dtype == ONNG_U8;
    const int rank = k + 1;      // one more, as the row itself may be a maximum
    P.nch = u8 ? nch_for(ONNG_U8, Q->dim) : (Q->dim + 31) / 32;
    // u8 above half a million base rows: the sweep in order of locality of
    // topk_u8_wide_kernel meets fewer candidates (k 100, ms: 400,000 rows 42.3,
    // here 35.8; 1M rows 170, here 234)
    if (u8 && nb > 500000) return P;
    // One row in f is sampled: the bound costs 1 / f of the filter's products and
    // lets about k f candidates through.  Measured (ms, k 100) at f = 2, 4, 8: f32
    // 33,000 rows 1.52, 1.77, 2.33; 100,003 6.21, 6.28, 7.47; 300,000 38.8, 39.8,
    // 45.6; 1M 396, 370, 392; u8 70,000 2.56, 3.51, 6.12; 400,000 37.7, 35.8, 45.3.
    int f = nb >= 350000 ? 4 : 2;
    for (; f >= 1; f /= 2) {
        const int64_t want = nb * 181 / 128 / f;         // pow2 within sqrt 2 of nb / f
        P.ns_log2 = 6;
        while ((2ll << P.ns_log2) <= std::min(want, nb)) P.ns_log2++;
        const int64_t need = (int64_t)(2.0 * k * (double)nb / (double)(1ll << P.ns_log2)) + 64;
        P.cap = 256;
        while (P.cap < need) P.cap *= 2;
        if (P.cap <= 2048) break;
    }
    if (f < 1) return P;
    const int64_t tiles = (1ll << P.ns_log2) / BN;
    int want_groups = 512;
    while (want_groups < 8 * rank) want_groups *= 2;
    want_groups = std::min(want_groups, 2048);
    P.group_tiles = 1;
    while (tiles / P.group_tiles * 16 > want_groups) P.group_tiles *= 2;
    P.groups = (int)(tiles / P.group_tiles * 16);
    if (P.groups < 2 * rank) return P;
    const int64_t chunks = (Q->n + WB_CHUNK - 1) / WB_CHUNK;
    const int64_t row_blocks = ((Q->n + chunks - 1) / chunks + WB_ROWS - 1) / WB_ROWS;
    P.chunk = row_blocks * WB_ROWS;
    const int64_t resident = 3 * (int64_t)device_cu_count();
    const int64_t ntiles[2] = {tiles, (nb + BN - 1) / BN};
    for (int m = 0; m < 2; m++) {
        const int64_t unit = m == 0 ? P.group_tiles : 1;
        const int64_t units = (ntiles[m] + unit - 1) / unit;
        int64_t best_cost = INT64_MAX;
        const int64_t top = std::min(units, std::max<int64_t>(1, 4 * resident / row_blocks));
        for (int64_t sp = 1; sp <= top; sp++) {
            const int64_t per = (units + sp - 1) / sp * unit;
            const int64_t rounds = (row_blocks * ((ntiles[m] + per - 1) / per) + resident - 1) / resident;
            const int64_t cost = rounds * (per + 2);
            if (cost < best_cost) {
                best_cost = cost;
                P.per_split[m] = (int)per;
                P.splits[m] = (int)((ntiles[m] + per - 1) / per);
            }
        }
    }
    P.use = true;
    return P;
}

onng_status launch_wide_bound(const TopkArgs &t, const onng_vectors *Q, bool same_rows, const WidePlan &P,
                              const WideBufs &w, hipStream_t st) {
    const bool u8 = Q->dtype == ONNG_U8;
    const bool cosine = Q->metric == ONNG_COSINE;
    WideArgs A;
    A.t = t;
    const int pitch = P.nch * 64;
    if (!u8) {
        hipLaunchKernelGGL(len_zero_kernel, dim3(1), dim3(2), 0, st, w.len);
        hipLaunchKernelGGL(len_max_kernel, dim3(256), dim3(256), 0, st, static_cast<const float *>(t.bn), t.nb, w.len);
        hipLaunchKernelGGL(len_max_kernel, dim3(256), dim3(256), 0, st, static_cast<const float *>(t.qn), t.nq, w.len + 1);
    }
    auto convert = [&](const uint8_t *src, int64_t sp, int64_t n, uint8_t *dst) {
        const dim3 g((unsigned)((n * (pitch / 16) + 255) / 256)), bl(256);
        if (u8) hipLaunchKernelGGL(to_i8_kernel, g, bl, 0, st, src, sp, n, t.dim, dst, pitch);
        else hipLaunchKernelGGL(to_f16_kernel, g, bl, 0, st, src, sp, n, t.dim, w.len, dst, pitch);
    };
    convert(t.b, t.b_pitch, t.nb, w.bh);
    if (!same_rows) convert(t.q, t.q_pitch, t.nq, w.qh);
    A.t.b = w.bh;
    A.t.q = same_rows ? w.bh : w.qh;
    A.t.b_pitch = A.t.q_pitch = pitch;
    A.side = static_cast<const uint32_t *>(t.bn);
    if (!u8 && !cosine) {
        hipLaunchKernelGGL(side_f32_kernel, dim3((unsigned)((t.nb + 255) / 256)), dim3(256), 0, st,
                           static_cast<const float *>(t.bn), t.nb, w.len, w.side);
        A.side = reinterpret_cast<const uint32_t *>(w.side);
    }
    A.ns_log2 = P.ns_log2;
    A.group_tiles = P.group_tiles;
    A.groups = P.groups;
    A.mins = w.mins;
    A.tau = w.tau;
    A.cnt = w.cnt;
    A.cand = w.cand;
    A.cap = P.cap;
    A.len = w.len;
    const int rank = t.k + (t.exclude_self ? 1 : 0);
    // Self exclusion: the passes leave out the column that is the row's place, which
    // in a candidate list is not its id.  There the own id goes at the end, from the
    // few candidates (read and compared where the passes queue them it cost a table
    // of 70,000 u8 rows, without a list, 25 of 2476 us).
    const bool drop_own = t.exclude_self && t.b_ids;
    if (drop_own) A.t.exclude_self = 0;
    A.drop_own = drop_own;
    // no D reaches this bound: u8 lim INT32_MAX - 1; f32 lim +inf (~ its sort key)
    const uint32_t none = u8 ? 0u : ~0xFF800000u;
    for (int64_t r0 = 0; r0 < t.nq; r0 += P.chunk) {
        A.row0 = r0;
        A.rows = (int32_t)std::min<int64_t>(P.chunk, t.nq - r0);
        for (int m = 0; m < 2; m++) {
            const bool bound = m == 0;
            const void *fn = u8 ? (bound ? wide_fn<ONNG_U8, ONNG_L2SQ, true>(P.nch) : wide_fn<ONNG_U8, ONNG_L2SQ, false>(P.nch))
                             : cosine ? (bound ? wide_fn<ONNG_F32, ONNG_COSINE, true>(P.nch) : wide_fn<ONNG_F32, ONNG_COSINE, false>(P.nch))
                                      : (bound ? wide_fn<ONNG_F32, ONNG_L2SQ, true>(P.nch) : wide_fn<ONNG_F32, ONNG_L2SQ, false>(P.nch));
            const size_t lds = wide_lds(pitch, !bound);
            ONNG_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            A.t.tiles_per_split = P.per_split[m];
            void *args[] = {&A};
            ONNG_HIP(hipLaunchKernel(fn, dim3((unsigned)((A.rows + WB_ROWS - 1) / WB_ROWS), (unsigned)P.splits[m]),
                                     dim3(256), args, lds, st));
            if (bound)
                launch_bound_select(w.mins, A.rows, P.groups, rank, bound_most(P.cap, P.ns_log2, t.nb), 31, u8 ? 0 : 8,
                                    P.cap, 0, none, w.tau, w.cnt, r0 == 0 ? w.redo : nullptr, st);
        }
        if (u8) {
            launch_bound_sort(true, w.cand, P.cap, w.cnt, A.rows, t.k, drop_own, t.out_ids, t.out_d, w.redo, r0, st);
        } else {
            const void *ff = cosine ? finish_fn<ONNG_COSINE>(P.cap) : finish_fn<ONNG_L2SQ>(P.cap);
            const size_t fl = (size_t)P.cap * 8 + WAVE * FIN_PITCH + 512;
            const uint8_t *qp = t.q, *bp = t.b;
            int64_t qpi = t.q_pitch, bpi = t.b_pitch;
            int32_t *redo = w.redo;
            void *fargs[] = {&A, &qp, &qpi, &bp, &bpi, &redo};
            ONNG_HIP(hipFuncSetAttribute(ff, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fl));
            ONNG_HIP(hipLaunchKernel(ff, dim3((unsigned)A.rows), dim3(WAVE), fargs, fl, st));
        }
    }
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

}  // namespace topk_detail
}  // namespace onng
