// Exact rerank of per-query candidate pools: distances recomputed from the
// given rows (f32 or f64 accumulation) and the k best (distance, id) kept.
// Used for the ground truth of float data (f32 screening, then f64) and for
// re-scoring low-precision search results from f32 rows.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "dist.h"
#include "onng_internal.h"
#include "wave.h"

namespace onng {

namespace {

constexpr int MAXPOOL = 1024;

__device__ __forceinline__ double elem_at(const uint8_t *row, int dtype, int c, float sc) {
    switch (dtype) {
    case ONNG_U8: return (double)row[c];
    case ONNG_F32: return (double)reinterpret_cast<const float *>(row)[c];
    case ONNG_F16: return (double)(float)__builtin_bit_cast(_Float16, reinterpret_cast<const uint16_t *>(row)[c]);
    case ONNG_BF16: return (double)__uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(row)[c] << 16);
    default: return (double)fp8_to_f32(row[c]) * (double)sc;
    }
}

template <int CTRL>
__device__ __forceinline__ double dpp64(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    return __builtin_bit_cast(double, (uint64_t)dpp<CTRL>((uint32_t)(u >> 32)) << 32 | dpp<CTRL>((uint32_t)u));
}

template <typename T>
__device__ __forceinline__ T plus_ror8(T x) { return x + (sizeof(T) == 8 ? (T)dpp64<DPP_ROW_ROR8>(x) : (T)dpp<DPP_ROW_ROR8>((float)x)); }
template <typename T>
__device__ __forceinline__ T plus_ror4(T x) { return x + (sizeof(T) == 8 ? (T)dpp64<DPP_ROW_ROR4>(x) : (T)dpp<DPP_ROW_ROR4>((float)x)); }
template <typename T>
__device__ __forceinline__ T plus_xor2(T x) { return x + (sizeof(T) == 8 ? (T)dpp64<DPP_QP_2301>(x) : (T)dpp<DPP_QP_2301>((float)x)); }
template <typename T>
__device__ __forceinline__ T plus_xor1(T x) { return x + (sizeof(T) == 8 ? (T)dpp64<DPP_QP_1032>(x) : (T)dpp<DPP_QP_1032>((float)x)); }

// One block per query.  Sixteen lanes share a pool row, four consecutive
// components each per 64, and RR_ROWS rows of a lane group are in flight (RR_AHEAD,
// or one where the lane groups hold the pool at once); then
// every entry's place is the number of entries before it under (d, id).
// Bound by the random row reads: the pool's rows once.  The sum of a row is
// the tree of one component per lane (chains over components 64 apart, then
// lanes 32, 16, .. 1 apart), kept as it was when one row at a time took the
// whole wave, so f32 distances and their ties are unchanged.  10,000 queries
// x 74 rows of 100 f32, f64 sums: 113 us; one row at a time 527 us.
constexpr int RR_AHEAD = 4;

template <bool F64, bool PLAIN_F32, int RR_ROWS>
__global__ void __launch_bounds__(256) rerank_kernel(const uint8_t *q, int64_t qp, int qdt,
                                                     const float *qsc, const uint8_t *b,
                                                     int64_t bp, int bdt, const float *bsc,
                                                     int dim, int metric, const int32_t *pool,
                                                     int psz, int k, int32_t *out_ids,
                                                     void *out_d) {
    typedef typename std::conditional<F64, double, float>::type acc_t;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    double *dd = reinterpret_cast<double *>(smem);
    int32_t *di = reinterpret_cast<int32_t *>(dd + psz);
    const int64_t qi = blockIdx.x;
    const uint8_t *qr = q + qi * qp;
    const float qs = qsc ? qsc[qi] : 1.0f;
    const int sub = threadIdx.x & 15;
    const int groups = blockDim.x / 16;
    // four components at c, zero past dim; PLAIN_F32 rows are 16-byte aligned
    // and padded to it, and what the padding holds is masked
    auto four = [&](const uint8_t *row, int dt, float sc, int c, acc_t *v) {
        if constexpr (PLAIN_F32) {
            float4 f = {0.0f, 0.0f, 0.0f, 0.0f};
            if (c < dim) f = *reinterpret_cast<const float4 *>(row + (int64_t)c * 4);
            v[0] = f.x;
            v[1] = c + 1 < dim ? f.y : 0.0f;
            v[2] = c + 2 < dim ? f.z : 0.0f;
            v[3] = c + 3 < dim ? f.w : 0.0f;
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = c + e < dim ? (acc_t)elem_at(row, dt, c + e, sc) : (acc_t)0;
        }
    };
    for (int i0 = threadIdx.x / 16; i0 < psz; i0 += groups * RR_ROWS) {
        int32_t id[RR_ROWS];
        const uint8_t *br[RR_ROWS];
        float bs[RR_ROWS];
        acc_t acc[RR_ROWS][4];
#pragma unroll
        for (int r = 0; r < RR_ROWS; r++) {
            const int i = i0 + r * groups;
            id[r] = i < psz ? pool[qi * psz + i] : -1;
            br[r] = b + (int64_t)max(id[r], 0) * bp;
            bs[r] = bsc && id[r] >= 0 ? bsc[id[r]] : 1.0f;
#pragma unroll
            for (int e = 0; e < 4; e++) acc[r][e] = 0;
        }
        for (int c = 4 * sub; c < dim; c += 64) {
            acc_t x[RR_ROWS][4], y[4];
#pragma unroll
            for (int r = 0; r < RR_ROWS; r++)
                if (id[r] >= 0) four(br[r], bdt, bs[r], c, x[r]);
                else x[r][0] = x[r][1] = x[r][2] = x[r][3] = 0;
            four(qr, qdt, qs, c, y);
#pragma unroll
            for (int r = 0; r < RR_ROWS; r++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    if (c + e >= dim) continue;
                    if (metric == ONNG_L2SQ) {
                        const acc_t df = x[r][e] - y[e];
                        acc[r][e] = F64 ? (acc_t)(acc[r][e] + df * df) : (acc_t)fmaf(df, df, acc[r][e]);
                    } else {
                        acc[r][e] = F64 ? (acc_t)(acc[r][e] + x[r][e] * y[e])
                                        : (acc_t)fmaf(x[r][e], y[e], acc[r][e]);
                    }
                }
        }
#pragma unroll
        for (int r = 0; r < RR_ROWS; r++) {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                // components 32, 16, 8 and 4 apart: lanes 8, 4, 2, 1 apart
                acc_t t = acc[r][e];
                t = plus_ror8(t);
                t = plus_ror4(t);
                t = plus_xor2(t);
                acc[r][e] = plus_xor1(t);
            }
            const acc_t sum = (acc[r][0] + acc[r][2]) + (acc[r][1] + acc[r][3]);
            const int i = i0 + r * groups;
            if (sub == 0 && i < psz) {
                const acc_t d = metric == ONNG_COSINE ? (acc_t)1 - sum : sum;
                dd[i] = id[r] >= 0 ? (double)d : __builtin_inf();
                di[i] = id[r];
            }
        }
    }
    __syncthreads();
    // rank of each entry under (d, id) with missing ids last
    for (int i = threadIdx.x; i < psz; i += blockDim.x) {
        const double d = dd[i];
        const int32_t id = di[i];
        if (id < 0) continue;
        int rank = 0;
        for (int j = 0; j < psz; j++) {
            const double dj = dd[j];
            const int32_t ij = di[j];
            rank += ij >= 0 && (dj < d || (dj == d && ij < id));
        }
        if (rank < k) {
            out_ids[qi * k + rank] = id;
            if (F64) reinterpret_cast<double *>(out_d)[qi * k + rank] = d;
            else reinterpret_cast<float *>(out_d)[qi * k + rank] = (float)d;
        }
    }
    // pad
    int valid = 0;
    for (int j = 0; j < psz; j++) valid += di[j] >= 0;
    for (int i = valid + threadIdx.x; i < k; i += blockDim.x) {
        out_ids[qi * k + i] = -1;
        if (F64) reinterpret_cast<double *>(out_d)[qi * k + i] = __builtin_inf();
        else reinterpret_cast<float *>(out_d)[qi * k + i] = __builtin_inff();
    }
}

}  // namespace

onng_status rerank_launch(const onng_vectors *Q, const onng_vectors *B, const int32_t *pool,
                          int32_t psz, int32_t k, int32_t use_f64, int32_t *ids, void *dists,
                          hipStream_t st) {
    if (psz > MAXPOOL) {
        set_error("onng_rerank: pool_size above 1024");
        return ONNG_ERR_UNSUPPORTED;
    }
    if (Q->n == 0) return ONNG_OK;
    const bool plain = Q->dtype == ONNG_F32 && B->dtype == ONNG_F32;
    auto pick = [&](auto ahead) {
        constexpr int R = decltype(ahead)::value;
        return use_f64 ? (plain ? rerank_kernel<true, true, R> : rerank_kernel<true, false, R>)
                       : (plain ? rerank_kernel<false, true, R> : rerank_kernel<false, false, R>);
    };
    // a pool of at most four rows fills no second row of a lane group (40,000 queries
    // x 1 row of 8 f32, f64 sums: 27.7 us with four rows ahead, 14.4 with one; a
    // wave to a row 25.0)
    auto fn = psz <= 4 ? pick(std::integral_constant<int, 1>()) : pick(std::integral_constant<int, RR_AHEAD>());
    // one wave per query once the queries alone fill the chip (32 waves on each
    // compute unit), else up to four that share its rows
    int waves = 1;
    while (waves < 4 && Q->n * waves * 2 <= (int64_t)32 * device_cu_count() &&
           psz > waves * 4 * RR_AHEAD)
        waves *= 2;
    hipLaunchKernelGGL(fn, dim3((unsigned)Q->n), dim3(waves * WAVE), (size_t)psz * 12, st,
                       static_cast<const uint8_t *>(Q->data), Q->pitch_bytes, Q->dtype, Q->scale,
                       static_cast<const uint8_t *>(B->data), B->pitch_bytes, B->dtype, B->scale,
                       Q->dim, Q->metric, pool, psz, k, ids, dists);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

}  // namespace onng
