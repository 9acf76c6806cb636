// Low-precision storage of f32 rows: f16 and bf16 (round to nearest even),
// and OCP fp8 e4m3fn with a per-row f32 scale (nearest even, saturating).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "onng_internal.h"
#include "wave.h"

namespace onng {

namespace {

__device__ __forceinline__ uint32_t f32_to_bf16(float x) {
    uint32_t b = __float_as_uint(x);
    if ((b & 0x7fffffffu) > 0x7f800000u) return (b >> 16) | 0x40u;   // NaN stays NaN
    b += 0x7fffu + ((b >> 16) & 1u);
    return b >> 16;
}

__device__ __forceinline__ uint32_t f32_to_f16(float x) {
    _Float16 h = (_Float16)x;   // v_cvt_f16_f32, round to nearest even
    return __builtin_bit_cast(uint16_t, h);
}

// e4m3fn: bias 7, largest finite 448 = 1.75 * 2^8, smallest normal 2^-6,
// subnormal spacing 2^-9; S.1111.111 is NaN.
__device__ __forceinline__ uint32_t f32_to_fp8(float x) {
    uint32_t sign = (__float_as_uint(x) >> 31) << 7;
    if (__builtin_isnan(x)) return sign | 0x7fu;
    float a = fabsf(x);
    if (!(a < 448.0f)) return sign | 0x7eu;                 // saturate
    if (a < 0x1p-6f) {
        uint32_t m = (uint32_t)rintf(a * 0x1p9f);          // exact scaling, then RNE
        return sign | m;                                   // m == 8 is the smallest normal
    }
    int e;
    frexpf(a, &e);
    int E = e - 1;                                         // a in [2^E, 2^(E+1))
    float mant = rintf(ldexpf(a, 3 - E));                  // in [8, 16]
    uint32_t M = (uint32_t)mant;
    if (M == 16u) { M = 8u; E += 1; }
    if (E > 8) return sign | 0x7eu;
    return sign | ((uint32_t)(E + 7) << 3) | (M - 8u);
}

// The general form: any alignment, one element at a time, a wave per row.
__global__ void encode_kernel(const float *src, int64_t n, int dim, int dtype, uint8_t *dst,
                              int64_t pitch, float *scale) {
    int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    int lane = threadIdx.x & 63;
    if (row >= n) return;
    const float *x = src + row * dim;
    uint8_t *out = dst + row * pitch;
    float s = 1.0f;
    if (dtype == ONNG_FP8_E4M3) {
        float mx = 0.0f;
        for (int c = lane; c < dim; c += 64) mx = fmaxf(mx, fabsf(x[c]));
        for (int m = 32; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m));
        s = mx > 0.0f ? __fdiv_rn(mx, 448.0f) : 1.0f;
        if (lane == 0) {
            if (scale) scale[row] = s;
            else *reinterpret_cast<float *>(out + pitch - 4) = s;   // in the row's tail
        }
    }
    int esz = dtype == ONNG_F32 ? 4 : (dtype == ONNG_F16 || dtype == ONNG_BF16) ? 2 : 1;
    const int64_t fill = dtype == ONNG_FP8_E4M3 && !scale ? pitch - 4 : pitch;
    for (int64_t c = lane; c * esz < fill; c += 64) {
        if (c >= dim) {
            for (int b = 0; b < esz; b++) out[c * esz + b] = 0;
            continue;
        }
        float v = x[c];
        switch (dtype) {
        case ONNG_F32: reinterpret_cast<float *>(out)[c] = v; break;
        case ONNG_F16: reinterpret_cast<uint16_t *>(out)[c] = (uint16_t)f32_to_f16(v); break;
        case ONNG_BF16: reinterpret_cast<uint16_t *>(out)[c] = (uint16_t)f32_to_bf16(v); break;
        default: out[c] = (uint8_t)f32_to_fp8(__fdiv_rn(v, s)); break;
        }
    }
}

// Four consecutive elements per lane: one store of 4 (fp8), 8 (f16, bf16) or
// 16 bytes (f32).
template <int DT>
__device__ __forceinline__ void put4(uint8_t *at, float4 v, float s) {
    if constexpr (DT == ONNG_F32) {
        *reinterpret_cast<float4 *>(at) = v;
    } else if constexpr (DT == ONNG_F16) {
        *reinterpret_cast<uint2 *>(at) = uint2{f32_to_f16(v.x) | f32_to_f16(v.y) << 16,
                                               f32_to_f16(v.z) | f32_to_f16(v.w) << 16};
    } else if constexpr (DT == ONNG_BF16) {
        *reinterpret_cast<uint2 *>(at) = uint2{f32_to_bf16(v.x) | f32_to_bf16(v.y) << 16,
                                               f32_to_bf16(v.z) | f32_to_bf16(v.w) << 16};
    } else {
        const float q[4] = {__fdiv_rn(v.x, s), __fdiv_rn(v.y, s), __fdiv_rn(v.z, s), __fdiv_rn(v.w, s)};
        uint32_t w;
        if (q[0] != q[0] || q[1] != q[1] || q[2] != q[2] || q[3] != q[3]) {
            w = f32_to_fp8(q[0]) | f32_to_fp8(q[1]) << 8 | f32_to_fp8(q[2]) << 16 | f32_to_fp8(q[3]) << 24;
        } else {
            // the conversion instruction rounds to nearest even; out of range
            // it would give NaN, so the values saturate first
            float c[4];
#pragma unroll
            for (int e = 0; e < 4; e++) c[e] = fminf(fmaxf(q[e], -448.0f), 448.0f);
            int pk = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], 0, false);
            pk = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], pk, true);
            w = (uint32_t)pk;
        }
        *reinterpret_cast<uint32_t *>(at) = w;
    }
}

// max over the LPR lanes of a row
template <int LPR>
__device__ __forceinline__ float row_max(float x) {
    x = fmaxf(x, dpp<DPP_ROW_ROR8>(x));
    x = fmaxf(x, dpp<DPP_ROW_ROR4>(x));
    x = fmaxf(x, dpp<DPP_QP_2301>(x));
    x = fmaxf(x, dpp<DPP_QP_1032>(x));
    x = fmaxf(x, swz_xor<16>(x));
    return LPR == 64 ? fmaxf(x, __shfl_xor(x, 32)) : x;
}

// LPR lanes per row, four elements per lane and step; they take ROWS rows, whose
// loads are in flight together.  Bound by memory: it reads 4 dim bytes a row and
// writes the row.  Needs the destination aligned for put4; SRC4: the source rows
// are 16-byte aligned (else element loads).  Half a wave and four rows (1M x 100 to
// fp8 rows with the scale in the row: 106 us, 512 MB, the rate of a large copy; one
// element per lane and byte stores: 383 us); a wave a row for rows of more steps.
template <int DT, bool SRC4, int LPR, int ROWS>
__global__ void __launch_bounds__(256) encode4_kernel(const float *src, int64_t n, int dim,
                                                      uint8_t *dst, int64_t pitch, float *scale) {
    constexpr int ESZ = DT == ONNG_F32 ? 4 : DT == ONNG_FP8_E4M3 ? 1 : 2;
    const int64_t row0 = ((int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR) * ROWS;
    const int l = threadIdx.x & (LPR - 1);
    const int64_t fill = DT == ONNG_FP8_E4M3 && !scale ? pitch - 4 : pitch;
    auto load = [&](int64_t row, int c) {
        const float *x = src + row * dim + c;
        float4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row >= n || c >= dim) return v;
        if (SRC4) return *reinterpret_cast<const float4 *>(x);   // dim is a multiple of 4
        v.x = x[0];
        if (c + 1 < dim) v.y = x[1];
        if (c + 2 < dim) v.z = x[2];
        if (c + 3 < dim) v.w = x[3];
        return v;
    };
    float4 v[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; r++) v[r] = load(row0 + r, 4 * l);
    float s[ROWS];
    auto max4 = [](float4 u) { return fmaxf(fmaxf(fabsf(u.x), fabsf(u.y)), fmaxf(fabsf(u.z), fabsf(u.w))); };
    if constexpr (DT == ONNG_FP8_E4M3) {
#pragma unroll
        for (int r = 0; r < ROWS; r++) s[r] = fmaxf(max4(v[r]), 0.0f);   // NaN elements do not count
        for (int c = 4 * (l + LPR); c < dim; c += 4 * LPR) {
            float4 u[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; r++) u[r] = load(row0 + r, c);
#pragma unroll
            for (int r = 0; r < ROWS; r++) s[r] = fmaxf(s[r], max4(u[r]));
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; r++) {
        if constexpr (DT != ONNG_FP8_E4M3) {
            s[r] = 1.0f;
        } else {
            const float mx = row_max<LPR>(s[r]);
            s[r] = mx > 0.0f ? __fdiv_rn(mx, 448.0f) : 1.0f;
            if (l == 0 && row0 + r < n) {
                if (scale) scale[row0 + r] = s[r];
                else *reinterpret_cast<float *>(dst + (row0 + r) * pitch + pitch - 4) = s[r];
            }
        }
    }
    // elements at or past dim are zero: the code of 0 is 0 in every type
#pragma unroll
    for (int r = 0; r < ROWS; r++)
        if (row0 + r < n && 4 * l * ESZ < fill) put4<DT>(dst + (row0 + r) * pitch + 4 * l * ESZ, v[r], s[r]);
    for (int64_t c = 4 * (l + LPR); c * ESZ < fill; c += 4 * LPR) {
        float4 u[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; r++) u[r] = load(row0 + r, (int)min<int64_t>(c, dim));
#pragma unroll
        for (int r = 0; r < ROWS; r++)
            if (row0 + r < n) put4<DT>(dst + (row0 + r) * pitch + c * ESZ, u[r], s[r]);
    }
}

}  // namespace

onng_status encode_launch(const float *src, int64_t n, int32_t dim, int32_t dtype, void *dst,
                          int64_t pitch, float *scale, hipStream_t st) {
    if (n == 0) return ONNG_OK;
    // put4 stores 4 elements at once; rows of another alignment take the general form
    const int unit = 4 * elem_bytes(dtype);
    if (reinterpret_cast<uintptr_t>(dst) % unit == 0 && pitch % unit == 0) {
        const bool s4 = reinterpret_cast<uintptr_t>(src) % 16 == 0 && dim % 4 == 0;
        // Rows of more than one step of half a wave take a wave each: the rows side by
        // side in the steps cost more than they hide.  us, half waves / so / one element
        // per lane: f32, 300,000 x 300: 192 / 130 / 175; fp8, 300,000 x 300: 120 / 132 /
        // 245, 93,750 x 960: 138 / 99 / 214, 1000 x 960: 16 / 9 / 11.  At 100 and 128
        // components: fp8, 900,000 x 100: 92 / 189 / 347.
        const bool wide = dim > 128;
        const int64_t per = wide ? 4 : 32;
        const dim3 grid((unsigned)((n + per - 1) / per)), block(256);
        uint8_t *d = static_cast<uint8_t *>(dst);
#define ONNG_ENC(DT)                                                                             \
    case DT: {                                                                                   \
        auto fn = wide ? (s4 ? encode4_kernel<DT, true, 64, 1> : encode4_kernel<DT, false, 64, 1>)  \
                       : (s4 ? encode4_kernel<DT, true, 32, 4> : encode4_kernel<DT, false, 32, 4>); \
        hipLaunchKernelGGL(fn, grid, block, 0, st, src, n, dim, d, pitch, scale);                \
        break;                                                                                   \
    }
        switch (dtype) {
            ONNG_ENC(ONNG_F32)
            ONNG_ENC(ONNG_F16)
            ONNG_ENC(ONNG_BF16)
            ONNG_ENC(ONNG_FP8_E4M3)
        }
#undef ONNG_ENC
    } else {
        hipLaunchKernelGGL(encode_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, src, n,
                           dim, dtype, static_cast<uint8_t *>(dst), pitch, scale);
    }
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

}  // namespace onng
