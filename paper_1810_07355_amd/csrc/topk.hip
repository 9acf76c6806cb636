// Exact top-k under (distance, id) by brute force on the matrix cores.
//
// The distance matrix is |x|^2 + |y|^2 - 2<x, y>; the dot products are the
// dense contraction and run on MFMA: int8 x int8 -> int32 (16x16x64) for u8
// data, after shifting every component by -128 (the shift cancels in x - y,
// and |<x', y'>| <= dim * 128^2 keeps int32 exact for dim <= 512), f32 x f32
// -> f32 (16x16x4)
// for float data.  Cosine distance on unit vectors is 1 - <x, y>.
//
// From 1024 base rows on, topk_bound.h's two passes do the work; topk_kernel
// here takes smaller bases, shapes whose sample or buffers would not fit, and the
// rows whose candidate buffer overflowed there or fell short of k.
// A block owns BM query rows (16 per wave) and sweeps the base rows in tiles
// of 64 staged in LDS.  Each row keeps its current k best keys sorted in LDS
// and a buffer of candidates that beat its k-th key; the buffer is sorted and
// merged into the list when it could overflow on the next tile, as soon as it
// holds k keys while the list is empty, and at the end.
// When the query rows alone give too few blocks to fill the chip (e.g. seed
// selection for one query batch), the base tiles are split among several
// blocks per row block, each writes its k best keys, and a second kernel
// merges them (the top k of the union of the parts' top k lists).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "onng_internal.h"
#include "topk_bound.h"
#include "topk_common.h"
#include "wave.h"

namespace onng {

using namespace topk_detail;

namespace {

// ---- per-row norms (int32 |x-128|^2 for u8, f32 |x|^2 otherwise) ----------
// |x|^2 of one row by a wave (u8: of x - 128)
__device__ __forceinline__ int32_t row_norm(const uint8_t *row, int dim, int32_t) {
    int32_t s = 0;
    for (int c = threadIdx.x & 63; c < dim; c += 64) {
        int v = (int)row[c] - 128;
        s += v * v;
    }
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
    return s;
}
__device__ __forceinline__ float row_norm(const uint8_t *row, int dim, float) {
    const float *r = reinterpret_cast<const float *>(row);
    float s = 0.0f;
    for (int c = threadIdx.x & 63; c < dim; c += 64) s = fmaf(r[c], r[c], s);
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
    return s;
}

template <typename T>
__global__ void norms_kernel(const uint8_t *x, int64_t pitch, int64_t n, int dim, T *out) {
    for (int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / 64; i < n; i += (int64_t)gridDim.x * 4) {
        const T s = row_norm(x + i * pitch, dim, T());
        if ((threadIdx.x & 63) == 0) out[i] = s;
    }
}

// A wave a row: the n candidate rows to dst, then the norms of the nq query
// rows, one launch for both: a single query's seeds and search 169.8 -> 167.9 us
// (in a stream of such calls; a launch by itself takes 4.5 us).
template <typename T>
__global__ void gather_norms_kernel(const uint8_t *src, int64_t pitch, const int32_t *ids, int64_t n,
                                    uint8_t *dst, const uint8_t *q, int64_t q_pitch, int64_t nq,
                                    int dim, T *qn) {
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (i < n) {
        const uint8_t *s = src + (int64_t)ids[i] * pitch;
        uint8_t *d = dst + i * pitch;
        for (int64_t c = lane * 16; c < pitch; c += 64 * 16)
            *reinterpret_cast<uint4 *>(d + c) = *reinterpret_cast<const uint4 *>(s + c);
    } else if (i < n + nq) {
        const T v = row_norm(q + (i - n) * q_pitch, dim, T());
        if (lane == 0) qn[i - n] = v;
    }
}

template <int DT, int MT, int NCH>
__global__ void __launch_bounds__(256) topk_kernel(TopkArgs a) {
    constexpr bool U8 = DT == ONNG_U8;
    constexpr int KQ = 4 * NCH;      // f32: components per k-group
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int wv = threadIdx.x / WAVE;
    const int nwaves = a.bm / 16;
    const int64_t row0 = (int64_t)blockIdx.x * a.bm;
    auto skip_row = [&](int64_t row) { return a.only && !a.only[1 + row]; };
    if (a.only) {
        if (!a.only[0]) return;
        const int64_t row = row0 + threadIdx.x;
        if (!__syncthreads_or((int)threadIdx.x < a.bm && row < a.nq && !skip_row(row))) return;
    }

    // LDS: [B tile][lists bm*kcap][cands bm*cb][tau bm][cnt bm][nlist bm][stage nwaves*64]
    char *p = smem;
    uint8_t *btile = reinterpret_cast<uint8_t *>(p);
    p += (size_t)BN * a.lds_pitch;
    uint64_t *lists = reinterpret_cast<uint64_t *>(p);
    p += (size_t)a.bm * a.kcap * 8;
    uint64_t *cands = reinterpret_cast<uint64_t *>(p);
    p += (size_t)a.bm * a.cb * 8;
    uint64_t *tau = reinterpret_cast<uint64_t *>(p);
    p += (size_t)a.bm * 8;
    int32_t *cnt = reinterpret_cast<int32_t *>(p);
    p += (size_t)a.bm * 4;
    int32_t *nlist = reinterpret_cast<int32_t *>(p);
    p += (size_t)a.bm * 4;
    uint64_t *stage = reinterpret_cast<uint64_t *>(p) + wv * WAVE;
    p += (size_t)nwaves * WAVE * 8;
    // per tile: base norms and global ids of its 64 rows, when needed
    uint32_t *t_norm = reinterpret_cast<uint32_t *>(p);
    if (a.side_norms) p += BN * 4;
    uint32_t *t_gid = reinterpret_cast<uint32_t *>(p);

    for (int i = threadIdx.x; i < a.bm; i += blockDim.x) {
        tau[i] = KEY_MAX;
        cnt[i] = 0;
        nlist[i] = 0;
    }

    // ---- this wave's 16 query rows as MFMA A operands ----
    const int arow = lane & 15;      // row within the wave's block
    const int kg = lane >> 4;        // k-group of this lane
    const int64_t qrow = row0 + wv * 16 + arow;
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
    // norms of the 4 output rows this lane sees in C (rows 4*kg + r)
    int32_t qn8[4] = {0, 0, 0, 0};
    float qnf[4] = {0, 0, 0, 0};
    int64_t crow[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
        crow[r] = row0 + wv * 16 + 4 * kg + r;
        if (crow[r] < a.nq) {
            if constexpr (U8) qn8[r] = reinterpret_cast<const int32_t *>(a.qn)[crow[r]];
            else if constexpr (MT == ONNG_L2SQ) qnf[r] = reinterpret_cast<const float *>(a.qn)[crow[r]];
        }
    }
    __syncthreads();

    auto flush_row = [&](int lr) {
        // lr: row within block; whole wave participates
        int n = uni(cnt[lr]);
        if (n == 0) return;
        uint64_t *lst = lists + (size_t)lr * a.kcap;
        int nl = uni(nlist[lr]);
        if (a.kcap <= 16) {
            // short lists (k <= 16): the first kcap lanes hold the list (none
            // while it is empty), the other lanes candidates; one sort of the
            // 64 lanes, the first kcap stay (no merge through LDS)
            const int kl = a.kcap;
            for (int c0 = 0; c0 < n;) {
                const int lo = nl == 0 ? 0 : kl;
                uint64_t key = KEY_MAX;
                if (lane < lo) {
                    if (lane < nl) key = lst[lane];
                } else if (c0 + lane - lo < n) {
                    key = cands[(size_t)lr * a.cb + c0 + lane - lo];
                }
                key = wave_sort(key, WAVE);
                nl = min(nl + min(WAVE - lo, n - c0), a.k);
                if (lane < kl) lst[lane] = key;
                wave_sync();
                c0 += WAVE - lo;
            }
            if (lane == 0) {
                cnt[lr] = 0;
                nlist[lr] = nl;
                tau[lr] = nl == a.k ? lst[a.k - 1] : KEY_MAX;
            }
            wave_sync();
            return;
        }
        for (int c0 = 0; c0 < n; c0 += WAVE) {
            uint64_t key = c0 + lane < n ? cands[(size_t)lr * a.cb + c0 + lane] : KEY_MAX;
            int nb = min(WAVE, n - c0);
            key = wave_sort(key, pow2_at_least(nb));
            int total = merge_sorted(lst, 0, nl, key, nb, a.k, stage, NoSpill());
            nl = min(total, a.k);
        }
        if (lane == 0) {
            cnt[lr] = 0;
            nlist[lr] = nl;
            tau[lr] = nl == a.k ? lst[a.k - 1] : KEY_MAX;
        }
        wave_sync();
    };

    const int ntiles = (int)((a.nb + BN - 1) / BN);
    constexpr int CPR = NCH * 4;     // 16-byte chunks of a staged row
    const int split = blockIdx.y;
    const int t_beg = split * a.tiles_per_split;
    const int t_end = min(ntiles, (split + 1) * a.tiles_per_split);
    // The next tile's rows are read into registers while the current tile is
    // computed (up to STG 16-byte chunks per thread), then stored to LDS.
    constexpr int STG = 9;
    constexpr int total = BN * CPR;
    const bool piped = total <= STG * (int)blockDim.x;
    uint4 stg[STG];
    uint32_t side_n = 0, side_g = 0;
    auto fetch_side = [&](int t) {
        const int64_t col = (int64_t)t * BN + threadIdx.x;
        side_n = 0;
        side_g = 0;
        if (threadIdx.x < BN && col < a.nb) {
            if (a.bn) side_n = reinterpret_cast<const uint32_t *>(a.bn)[col];
            if (a.b_ids) side_g = (uint32_t)a.b_ids[col];
        }
    };
    auto put_side = [&]() {
        if (threadIdx.x < BN) {
            if (a.bn) t_norm[threadIdx.x] = side_n;
            if (a.b_ids) t_gid[threadIdx.x] = side_g;
        }
    };
    // A thread's chunks sit at the same place in every tile; rows are read
    // with 32-bit offsets from the tile's first row.
    const uint32_t bp32 = (uint32_t)a.b_pitch;
    const int cmax = (int)min<int64_t>(CPR, a.b_pitch / 16);   // chunks a global row holds
    auto load_chunk = [&](const uint8_t *tb, int rows, int i) {
        const int r = i / CPR, c = i - r * CPR;
        if (r < rows && c < cmax)
            return *reinterpret_cast<const uint4 *>(tb + (uint32_t)r * bp32 + (uint32_t)c * 16u);
        return uint4{0, 0, 0, 0};
    };
    auto tile_rows = [&](int t) { return (int)min<int64_t>(BN, a.nb - (int64_t)t * BN); };
    auto tile_ptr = [&](int t) { return a.b + (int64_t)t * BN * a.b_pitch; };
    // Pipelined staging: thread chunk j is i = threadIdx.x + j * blockDim.x,
    // at global offset goff[j] in the tile and LDS offset loff[j] (low 24
    // bits; its chunk index within the row in the high 8).
    uint32_t goff[STG], loff[STG];
#pragma unroll
    for (int j = 0; j < STG; j++) {
        const int i = threadIdx.x + j * blockDim.x;
        const uint32_t r = (uint32_t)(i / CPR), c = (uint32_t)(i % CPR);
        goff[j] = r * bp32 + c * 16u;
        loff[j] = (r * (uint32_t)a.lds_pitch + c * 16u) | (c << 24);
    }
    const bool rows_long = cmax == CPR;
    auto fetch_tile = [&](int t) {
        fetch_side(t);
        const uint8_t *tb = tile_ptr(t);
        const int rows = tile_rows(t);
        if (rows == BN && rows_long) {
#pragma unroll
            for (int j = 0; j < STG; j++) {
                const int i = threadIdx.x + j * blockDim.x;
                if (i < total) stg[j] = *reinterpret_cast<const uint4 *>(tb + goff[j]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < STG; j++) {
                const int i = threadIdx.x + j * blockDim.x;
                stg[j] = i < total ? load_chunk(tb, rows, i) : uint4{0, 0, 0, 0};
            }
        }
    };
    // components at or past dim become 0 (a row's padding may hold anything)
    auto put_chunk_at = [&](uint32_t off, int c, uint4 v) {
        uint32_t w4[4] = {v.x, v.y, v.z, v.w};
        if constexpr (U8) {
            // x - 128 as int8 is x ^ 0x80
#pragma unroll
            for (int w = 0; w < 4; w++) w4[w] ^= 0x80808080u;
            if (c * 16 + 16 > a.dim) {
#pragma unroll
                for (int w = 0; w < 4; w++) {
                    const int valid = a.dim - (c * 16 + 4 * w);
                    if (valid <= 0) w4[w] = 0u;
                    else if (valid < 4) w4[w] &= (1u << (8 * valid)) - 1u;
                }
            }
        } else {
            if (c * 4 + 4 > a.dim) {
#pragma unroll
                for (int w = 0; w < 4; w++)
                    if (c * 4 + w >= a.dim) w4[w] = 0u;
            }
        }
        *reinterpret_cast<uint4 *>(btile + off) = uint4{w4[0], w4[1], w4[2], w4[3]};
    };
    auto put_chunk = [&](int i, uint4 v) {
        const int r = i / CPR, c = i - r * CPR;
        put_chunk_at((uint32_t)r * (uint32_t)a.lds_pitch + (uint32_t)c * 16u, c, v);
    };
    // For a kNN graph of rows in locality order the sweep starts at the row
    // block's own tile and wraps around: the nearest rows come first, so the
    // lists' thresholds are tight from the start and few later candidates
    // pass them.  The result does not depend on the order.
    const int rot0 = a.rotate ? (int)((row0 / BN) % ntiles) : 0;
    auto tile_at = [&](int i) { const int x = i + rot0; return x >= ntiles ? x - ntiles : x; };
    if (piped && t_beg < t_end) fetch_tile(tile_at(t_beg));
    for (int t = t_beg; t < t_end; t++) {
        const int tt = tile_at(t);
        const int64_t col0 = (int64_t)tt * BN;
        __syncthreads();
        // stage 64 base rows
        if (piped) {
#pragma unroll
            for (int j = 0; j < STG; j++) {
                const int i = threadIdx.x + j * blockDim.x;
                if (i < total) put_chunk_at(loff[j] & 0xFFFFFFu, (int)(loff[j] >> 24), stg[j]);
            }
            put_side();
        } else {
            fetch_side(tt);
            put_side();
            const uint8_t *tb = tile_ptr(tt);
            const int rows = tile_rows(tt);
            for (int i = threadIdx.x; i < total; i += blockDim.x) put_chunk(i, load_chunk(tb, rows, i));
        }
        __syncthreads();
        if (piped && t + 1 < t_end) fetch_tile(tile_at(t + 1));
        if (a.side_norms && !a.bn) {
            tile_norms<U8, CPR>(btile, a.lds_pitch, blockDim.x, t_norm);
            __syncthreads();
        }
        if (row0 + wv * 16 >= a.nq) continue;

        // ---- 16 query rows x 64 tile columns: four 16x16 blocks, their
        // accumulation chains interleaved ----
        const uint8_t *bbase = btile + arow * a.lds_pitch + (U8 ? kg * 16 : kg * KQ * 4);
        i32x4 acc8[4];
        f32x4 accf[4];
#pragma unroll
        for (int cb = 0; cb < 4; cb++) {
            acc8[cb] = i32x4{0, 0, 0, 0};
            accf[cb] = f32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int c = 0; c < NCH; c++) {
            if constexpr (U8) {
                i32x4 bv[4];
#pragma unroll
                for (int cb = 0; cb < 4; cb++)
                    bv[cb] = *reinterpret_cast<const i32x4 *>(bbase + cb * 16 * a.lds_pitch + c * 64);
#pragma unroll
                for (int cb = 0; cb < 4; cb++)
                    acc8[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A8[c], bv[cb], acc8[cb], 0, 0, 0);
            } else {
                f32x4 bv[4];
#pragma unroll
                for (int cb = 0; cb < 4; cb++)
                    bv[cb] = *reinterpret_cast<const f32x4 *>(bbase + cb * 16 * a.lds_pitch + c * 16);
#pragma unroll
                for (int j = 0; j < 4; j++)
#pragma unroll
                    for (int cb = 0; cb < 4; cb++)
                        accf[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(AF[4 * c + j], bv[cb][j],
                                                                          accf[cb], 0, 0, 0);
            }
        }

        // ---- epilogue: C layout, lane holds rows 4*kg + r of column arow
        // of each block.  A key can beat a row's list only if its distance
        // part is <= the high half of the row's threshold; that test alone
        // runs on every value, the full one on the few that pass it. ----
        uint64_t thr[4];      // 0 for rows past the end: no key is below it
        uint32_t thi[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const uint64_t tv = tau[wv * 16 + 4 * kg + r];
            thr[r] = crow[r] < a.nq ? tv : 0ull;
            thi[r] = (uint32_t)(thr[r] >> 32);
        }
        uint32_t dd[4][4];
        uint64_t hit[4];      // per block: lanes with a value that passed the prefilter
#pragma unroll
        for (int cb = 0; cb < 4; cb++) {
            int32_t bn8 = 0;
            float bnf = 0.0f;
            if constexpr (U8) bn8 = (int32_t)t_norm[cb * 16 + arow];
            else if constexpr (MT == ONNG_L2SQ) bnf = __uint_as_float(t_norm[cb * 16 + arow]);
            hit[cb] = 0;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                uint32_t dord;
                if constexpr (U8) {
                    dord = (uint32_t)(qn8[r] + bn8 - 2 * acc8[cb][r]);
                } else if constexpr (MT == ONNG_L2SQ) {
                    dord = ord_f32(qnf[r] + bnf - 2.0f * accf[cb][r]);
                } else {
                    dord = ord_f32(1.0f - accf[cb][r]);
                }
                dd[cb][r] = dord;
                hit[cb] |= ballot(dord <= thi[r]);
            }
        }
        const bool partial = col0 + BN > a.nb;
#pragma unroll
        for (int cb = 0; cb < 4; cb++) {
            if (!hit[cb]) continue;
            const int64_t col = col0 + cb * 16 + arow;
            const bool cok = !partial || col < a.nb;
            const uint32_t gid = a.b_ids ? t_gid[cb * 16 + arow] : (uint32_t)col;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const uint64_t key = make_key(dd[cb][r], gid);
                if (cok && key < thr[r] && !(a.exclude_self && (int64_t)gid == crow[r])) {
                    int lr = wv * 16 + 4 * kg + r;
                    int slot = atomicAdd(&cnt[lr], 1);
                    cands[(size_t)lr * a.cb + slot] = key;
                }
            }
        }
        wave_sync();
        // rows whose buffer could overflow on the next tile
        // (or, while its list is still empty, that already hold k keys: the
        // list then starts from the best k of the first tiles)
        const int cr = cnt[wv * 16 + (lane & 15)];
        const int nr = nlist[wv * 16 + (lane & 15)];
        uint64_t over = ballot(lane < 16 && (cr > a.cb - BN || (nr == 0 && cr >= a.k)));
        while (over) {
            const int r = __builtin_ctzll(over);
            over &= over - 1;
            flush_row(wv * 16 + r);
        }
    }
    __syncthreads();
    if (row0 + wv * 16 >= a.nq) return;
    for (int r = 0; r < 16; r++) {
        int lr = wv * 16 + r;
        int64_t grow = row0 + lr;
        if (grow >= a.nq) break;
        if (skip_row(grow)) continue;
        flush_row(lr);
        int nl = uni(nlist[lr]);
        const uint64_t *lst = lists + (size_t)lr * a.kcap;
        if (a.splits > 1) {
            uint64_t *dst = a.part + ((size_t)grow * a.splits + split) * a.k;
            for (int i = lane; i < a.k; i += WAVE) dst[i] = i < nl ? lst[i] : KEY_MAX;
            continue;
        }
        for (int i = lane; i < a.k; i += WAVE) {
            uint64_t key = i < nl ? lst[i] : KEY_MAX;
            a.out_ids[grow * a.k + i] = i < nl ? (int32_t)(uint32_t)key : -1;
            if constexpr (U8) {
                reinterpret_cast<int32_t *>(a.out_d)[grow * a.k + i] =
                    i < nl ? (int32_t)(key >> 32) : INT32_MAX;
            } else {
                reinterpret_cast<float *>(a.out_d)[grow * a.k + i] =
                    i < nl ? unord_f32((uint32_t)(key >> 32)) : __builtin_inff();
            }
        }
    }
}

// One wave per query row: the k best of the splits * k part keys.
template <bool U8>
__global__ void __launch_bounds__(256) merge_parts_kernel(const uint64_t *part, int64_t nq,
                                                          int splits, int k, int kcap,
                                                          int32_t *out_ids, void *out_d,
                                                          const int32_t *only) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int wv = threadIdx.x / WAVE;
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x / WAVE) + wv;
    if (row >= nq) return;
    if (only && (!only[0] || !only[1 + row])) return;
    uint64_t *lst = reinterpret_cast<uint64_t *>(smem) + (size_t)wv * (kcap + WAVE);
    uint64_t *stage = lst + kcap;
    const uint64_t *src = part + (size_t)row * splits * k;
    const int n = splits * k;
    int nl = 0;
    for (int c0 = 0; c0 < n; c0 += WAVE) {
        uint64_t key = c0 + lane < n ? src[c0 + lane] : KEY_MAX;
        key = wave_sort(key, WAVE);
        // KEY_MAX pads missing entries; they sort last
        int nb = __popcll(ballot(key != KEY_MAX));
        if (nb == 0) continue;
        nl = min(merge_sorted(lst, 0, nl, key, nb, k, stage, NoSpill()), k);
    }
    for (int i = lane; i < k; i += WAVE) {
        uint64_t key = i < nl ? lst[i] : KEY_MAX;
        out_ids[row * k + i] = i < nl ? (int32_t)(uint32_t)key : -1;
        if constexpr (U8)
            reinterpret_cast<int32_t *>(out_d)[row * k + i] = i < nl ? (int32_t)(key >> 32) : INT32_MAX;
        else
            reinterpret_cast<float *>(out_d)[row * k + i] =
                i < nl ? unord_f32((uint32_t)(key >> 32)) : __builtin_inff();
    }
}

// ---- between and after the passes of topk_bound.h ----
// One wave per row: an upper bound of the rank-th smallest of its group minima
// (the distances' low bits below `low` rounded up; `past` is added), and its
// counter cleared.  Bits are settled from `top` down by counting the minima at or
// below each trial value, VPL minima per lane in registers.  Where more than
// `most` minima are within the bound (equal distances; each minimum stands for
// nb / sampled rows), the candidates would overflow: the counter starts past the
// buffer, and with `none` for a bound nothing passes.  All rows equal, us: u8
// 70,000 x 128, k 100: 29,140 -> 10,100, f32 10,000 x 10,000 x 100, k 8: 970 -> 467
// (9,100 and 425 with the list kernel alone).
template <int VPL>
__global__ void __launch_bounds__(256) bound_select_kernel(const uint32_t *mins, int64_t nq, int groups,
                                                           int rank, int most, int top, int low, int cap,
                                                           uint32_t past, uint32_t none, uint32_t *tau,
                                                           int32_t *cnt, int32_t *clear) {
    const int64_t row = (int64_t)blockIdx.x * 4 + uni(threadIdx.x / WAVE);
    const int lane = lane_id();
    if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0;
    if (row >= nq) return;
    uint32_t x[VPL];
#pragma unroll
    for (int i = 0; i < VPL; i++) {
        const int g = i * WAVE + lane;
        x[i] = g < groups ? mins[row * groups + g] : ~0u;
    }
    uint32_t v = 0;
    int within = groups;   // minima within the bound: those of the last trial that held rank
    for (int bit = top; bit >= low; bit--) {
        const uint32_t trial = v | ((1u << bit) - 1u);
        int c = 0;
#pragma unroll
        for (int i = 0; i < VPL; i++) c += __popcll(ballot(x[i] <= trial));
        if (c < rank) v |= 1u << bit;
        else within = c;
    }
    if (lane == 0) {
        tau[row] = within > most ? none : (v | ((1u << low) - 1u)) + past;
        cnt[row] = within > most ? cap + 1 : 0;
    }
}

// One block per row: its cnt[row] candidates in order, the k first written.
// A row with more than `cap`, or with fewer than
// k (there are at least 1024 base rows, but the bound allows for one copy of the
// row itself and a candidate list may hold more), is left to the general kernel
// (redo[1 + row], and redo[0] for any).  Up to 64 candidates sort in registers,
// more by a bitonic network in LDS; with few rows the block has four waves.
// drop_own: candidates with the row's own id do not count.
template <bool U8>
__global__ void __launch_bounds__(256) bound_sort_kernel(const uint64_t *cand, int cap, const int32_t *cnt,
                                                         int k, int drop_own, int32_t *out_ids, void *out_d,
                                                         int32_t *redo, int64_t row0) {
    extern __shared__ __attribute__((aligned(16))) uint64_t sk[];
    const int64_t row = blockIdx.x;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int n = uni(cnt[row]);
    const uint64_t *src = cand + row * cap;
    auto is_own = [&](uint64_t key) { return drop_own && (int64_t)(uint32_t)key == row0 + row; };
    int own = 0;
    if (drop_own && n <= cap)
        for (int i0 = 0; i0 < n; i0 += nt) own += __syncthreads_count(i0 + tid < n && is_own(src[i0 + tid]));
    const bool bad = n > cap || n - own < k;
    if (tid == 0) redo[1 + row0 + row] = bad;
    if (bad) {
        if (tid == 0) redo[0] = 1;
        return;
    }
    auto put = [&](int i, uint64_t key) {
        const int64_t at = (row0 + row) * k + i;
        out_ids[at] = (int32_t)(uint32_t)key;
        if constexpr (U8) reinterpret_cast<int32_t *>(out_d)[at] = (int32_t)(key >> 32);
        else reinterpret_cast<float *>(out_d)[at] = unord_f32((uint32_t)(key >> 32));
    };
    if (n <= WAVE) {
        if (tid >= WAVE) return;
        uint64_t key = tid < n ? src[tid] : KEY_MAX;
        if (is_own(key)) key = KEY_MAX;
        key = wave_sort(key, pow2_at_least(n));
        if (tid < k) put(tid, key);
        return;
    }
    const int w = pow2_at_least(n);
    for (int i = tid; i < w; i += nt) sk[i] = i < n && !is_own(src[i]) ? src[i] : KEY_MAX;
    for (int size = 2; size <= w; size <<= 1)
        for (int d = size >> 1; d > 0; d >>= 1) {
            __syncthreads();
            for (int t = tid; t < w / 2; t += nt) {
                const int i = 2 * t - (t & (d - 1));   // lower of the pair (i, i + d)
                const uint64_t lo = sk[i], hi = sk[i + d];
                if ((lo > hi) == ((i & size) == 0)) sk[i] = hi, sk[i + d] = lo;
            }
        }
    __syncthreads();
    for (int i = tid; i < k; i += nt) put(i, sk[i]);
}

// Parts per row block.  With one block per compute unit (the LDS holds one
// block's tile, lists and buffers), the launch takes ceil(blocks / CUs)
// rounds, each as long as one part: about its tiles plus a few tiles' worth
// of list warm-up.  The part count minimises that product (parts keep at
// least 8 tiles).
int topk_splits(int64_t nq, int64_t nb, int bm) {
    const int64_t row_blocks = (nq + bm - 1) / bm;
    const int64_t ntiles = (nb + BN - 1) / BN;
    const int64_t cus = device_cu_count();
    if (row_blocks >= 4 * cus || ntiles < 16) return 1;
    const int64_t top = std::min<int64_t>(64, ntiles / 8);
    int64_t best = 1, best_cost = INT64_MAX;
    for (int64_t sp = 1; sp <= top; sp++) {
        const int64_t rounds = (row_blocks * sp + cus - 1) / cus;
        const int64_t cost = rounds * ((ntiles + sp - 1) / sp + 4);
        if (cost < best_cost) best = sp, best_cost = cost;
    }
    return (int)best;
}


template <int DT, int MT>
const void *topk_fn_for(int nch) {
    if constexpr (DT == ONNG_U8) {
        switch (nch) {
            case 1: return (const void *)topk_kernel<DT, MT, 1>;
            case 2: return (const void *)topk_kernel<DT, MT, 2>;
            case 4: return (const void *)topk_kernel<DT, MT, 4>;
            default: return (const void *)topk_kernel<DT, MT, 8>;
        }
    } else {
        switch (nch) {
            case 2: return (const void *)topk_kernel<DT, MT, 2>;
            case 4: return (const void *)topk_kernel<DT, MT, 4>;
            case 6: return (const void *)topk_kernel<DT, MT, 6>;
            case 7: return (const void *)topk_kernel<DT, MT, 7>;
            case 8: return (const void *)topk_kernel<DT, MT, 8>;
            case 12: return (const void *)topk_kernel<DT, MT, 12>;
            default: return (const void *)topk_kernel<DT, MT, 16>;
        }
    }
}

size_t topk_lds_bytes(int bm, int kcap, int cb, int lds_pitch, int side_words = 0) {
    int nwaves = bm / 16;
    return (size_t)BN * lds_pitch + (size_t)bm * kcap * 8 + (size_t)bm * cb * 8 + (size_t)bm * 16 +
           (size_t)nwaves * WAVE * 8 + (size_t)side_words * BN * 4;
}

// Query rows per block: 64 when the block's tile, lists and buffers fit in
// LDS, else 32.
int topk_side_words(int dtype, int metric, bool cand) {
    return (dtype == ONNG_U8 || metric == ONNG_L2SQ ? 1 : 0) + (cand ? 1 : 0);
}

int topk_bm(int32_t k, int dtype, int32_t dim, int side_words) {
    const int kcap = topk_kcap(k);
    const int lp = lds_pitch_for(dtype, dim);
    return kcap <= 128 && topk_lds_bytes(64, kcap, topk_cb(k), lp, side_words) <= 160 * 1024 ? 64
                                                                                            : 32;
}

// The f16-screened passes (and the bf16-screened list kernel behind them): f32 rows
// of at most 128 components, and so many queries that the list kernel's 128-row
// blocks fill the chip.  The line is the list kernel's; the passes, which split the
// columns among blocks, are faster below it too (kNN, 100 components, k 100, ms, the
// narrow passes / these: 9,000 rows 0.44 / 0.23, 32,000 rows 3.39 / 1.02).
bool topk_use_wide_f32(const onng_vectors *Q, int64_t nb, int32_t k) {
    return Q->dtype == ONNG_F32 && Q->dim <= FW_NCH * 32 && nb >= 16 * FW_BN &&
           Q->n >= (int64_t)FW_ROWS * device_cu_count() && fw_lds_bytes(topk_kcap(k)) <= 64 * 1024;
}

// The wide u8 passes and list kernel: the list kernel's 256-row blocks alone fill
// the chip (one per compute unit at least) and the rows fit two 64-byte k-steps.
bool topk_use_wide(const onng_vectors *Q, int64_t nb, int32_t k) {
    return Q->dtype == ONNG_U8 && nch_for(ONNG_U8, Q->dim) <= 2 && nb >= 16 * BN &&
           Q->n >= (int64_t)WIDE_ROWS * device_cu_count() &&
           wide_lds_bytes(lds_pitch_for(ONNG_U8, Q->dim), topk_kcap(k)) <= 64 * 1024;
}

// The bound-and-filter path (topk_bound.h): what it samples and how it is laid
// out, or use = false.
struct BoundPlan {
    bool use = false;
    int rw = 0;                  // row waves per block: 1, 4 or 8
    int64_t chunk = 0;           // query rows per launch
    int ns_log2 = 0, group_tiles = 0, quads = 0, groups = 0, cap = 0;
    int splits[2] = {1, 1}, per_split[2] = {0, 0};   // bound, filter
    size_t lds[2] = {0, 0};
};

BoundPlan topk_bound_plan(const onng_vectors *Q, int64_t nb, int32_t k) {
    BoundPlan P;
    const int rank = k + 1;      // one more, as the row itself may be a minimum
    // us at 1024 base rows, these passes / the list kernel: u8, k 8: 1 query 28 / 35,
    // 1000 queries 37 / 112; f32, k 100, 1 query 31 / 62 (from 17 queries on a sample of
    // so few rows does not serve k 100).  Below 1024 they would still win for small k
    // (u8, k 8, 1000 queries: 512 rows 35 / 104, 256 rows 36 / 82).
    if (Q->n < 1 || nb < 1024) return P;
    const int cw = Q->n <= 16 ? 4 : 1;
    P.rw = Q->n <= 16 ? 1 : Q->n <= 64 ? 4 : 8;
    // One row in f is sampled: the bound costs 1 / f of the filter's products
    // and lets about k f candidates through.  Measured (us) at f = 2, 4, 8: kNN of u8
    // rows, 128 components, k 10: 3000 rows 64, 66, 65; 10,007 154, 168, 184; 16,000 257,
    // 266, 297; 25,000 548, 528, 569; 50,000 1707, 1598, 1685 (k 100: f = 2 is ahead
    // throughout, 10,007 rows 261, 357, 815; 50,000 2459, 2727, 3369); of f32 rows, 100
    // components, k 10: 3000 rows 82, 78, 78; 10,007 388, 366, 366; 25,000 2253, 1876,
    // 1739 (k 100: 10,007 491, 554, 997; 25,000 2474, 2263, 2377); f32 100 x 1M x 96,
    // k 100: -, 369, 351; f32 10,000 x 200,000 x 100, k 74: -, 5746, 5313.
    int f = nb >= 65536 ? 8 : Q->dtype == ONNG_U8 && nb < 16384 ? 2 : 4;
    for (; f >= 1; f /= 2) {
        const int64_t want = nb * 181 / 128 / f;         // pow2 within sqrt 2 of nb / f
        P.ns_log2 = 6;
        while ((2ll << P.ns_log2) <= std::min(want, nb)) P.ns_log2++;
        int64_t need = (int64_t)(1.5 * k * (double)nb / (double)(1ll << P.ns_log2)) + 64;
        P.cap = 256;
        while (P.cap < need) P.cap *= 2;
        if (P.cap <= 4096 && Q->n * (int64_t)P.cap * 8 <= (1ll << 29)) break;
    }
    if (f < 1) return P;
    const int64_t ns = 1ll << P.ns_log2, tiles = ns / BN;
    int want_groups = 512;
    while (want_groups < 8 * rank) want_groups *= 2;
    want_groups = std::min(want_groups, 2048);
    // Query rows in equal chunks, so that candidates and group minima (at most
    // 1024 and 2048 per row where there is more than one chunk) stay within 1 GiB.
    const int bm = P.rw * 16;
    const int64_t chunks = (Q->n + BOUND_CHUNK - 1) / BOUND_CHUNK;
    const int64_t row_blocks = ((Q->n + chunks - 1) / chunks + bm - 1) / bm;
    P.chunk = row_blocks * bm;
    P.group_tiles = 1;
    while (tiles / P.group_tiles * 16 * cw > want_groups) P.group_tiles *= 2;
    // few row blocks: groups of fewer tiles, the minima of four lanes together,
    // so that more blocks share the sample
    if (P.group_tiles >= 4 && tiles / P.group_tiles * row_blocks < 2 * device_cu_count()) {
        P.group_tiles /= 4;
        P.quads = 1;
    }
    P.groups = (int)(tiles / P.group_tiles * 16 * cw) / (P.quads ? 4 : 1);
    if (P.groups < 2 * rank || P.groups > 2048) return P;
    for (int m = 0; m < 2; m++) P.lds[m] = bound_lds(lds_pitch_for(Q->dtype, Q->dim), P.rw, m == 1);
    if (P.lds[1] > 160 * 1024) return P;
    // Splits: all resident blocks (by LDS and by registers: four waves per SIMD,
    // three with RW = 4) run at once, so a launch takes ceil(blocks / resident)
    // rounds, each as long as one split and two tiles' worth of start and end.
    const int64_t ntiles[2] = {tiles, (nb + BN - 1) / BN};
    for (int m = 0; m < 2; m++) {
        const int64_t per_cu = std::min<int64_t>(160 * 1024 / (int64_t)P.lds[m], P.rw == 8 ? 2 : P.rw == 4 ? 3 : 4);
        const int64_t resident = std::max<int64_t>(per_cu, 1) * device_cu_count();
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

}  // namespace

namespace topk_detail {

void launch_bound_select(const uint32_t *mins, int64_t nq, int groups, int rank, int most, int top, int low,
                         int cap, uint32_t past, uint32_t none, uint32_t *tau, int32_t *cnt, int32_t *clear, hipStream_t st) {
    auto sel = groups <= 512 ? bound_select_kernel<8> : groups <= 1024 ? bound_select_kernel<16>
                                                                       : bound_select_kernel<32>;
    hipLaunchKernelGGL(sel, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, st, mins, nq, groups, rank, most,
                       top, low, cap, past, none, tau, cnt, clear);
}

void launch_bound_sort(bool u8, const uint64_t *cand, int cap, const int32_t *cnt, int64_t nq, int k,
                       bool drop_own, int32_t *ids, void *dists, int32_t *redo, int64_t row0, hipStream_t st) {
    auto fn = u8 ? bound_sort_kernel<true> : bound_sort_kernel<false>;
    hipLaunchKernelGGL(fn, dim3((unsigned)nq), dim3(nq < 1024 ? 256 : WAVE), (size_t)cap * 8, st, cand, cap,
                       cnt, k, (int)drop_own, ids, dists, redo, row0);
}

}  // namespace topk_detail

// Converted rows lie where the list kernel behind the passes, which starts when
// they are done, keeps its own: bh and qh are its bf16 copies of base and queries
// (f32), qh its candidate slots (u8; the base's rows have a place of their own).
static WideBufs carve_wide(Carver &c, const onng_vectors *Q, int64_t nb, const WidePlan &P, void *bh, void *qh) {
    WideBufs w{};
    if (!P.use) return w;
    const int64_t rows = std::min<int64_t>(Q->n, P.chunk);
    w.mins = c.take<uint32_t>((size_t)rows * P.groups);
    w.tau = c.take<uint32_t>(rows);
    w.cnt = c.take<int32_t>(rows);
    w.cand = c.take<uint64_t>((size_t)rows * P.cap);
    w.redo = c.take<int32_t>(Q->n + 1);
    static_assert(FW_NCH * 64 >= 4 * 64 && WIDE_CB * 8 >= 2 * 64, "room for a converted row");
    w.qh = static_cast<uint8_t *>(qh);
    if (Q->dtype == ONNG_U8) {
        w.bh = c.take<uint8_t>((size_t)nb * P.nch * 64);
    } else {
        w.bh = static_cast<uint8_t *>(bh);
        w.side = c.take<float>(nb);
        w.len = c.take<float>(2);
    }
    return w;
}

size_t topk_ws_size(const onng_vectors *Q, const onng_vectors *B, int64_t n_cand, int32_t k) {
    Carver c(nullptr);
    int64_t nb = n_cand > 0 ? n_cand : B->n;
    c.take<float>(Q->n);
    c.take<float>(nb);
    if (n_cand > 0) c.take<uint8_t>((size_t)nb * B->pitch_bytes);
    if (topk_use_wide(Q, nb, k)) {
        c.take<uint64_t>((size_t)Q->n * topk_kcap(k));
        c.take<uint64_t>((size_t)Q->n * WIDE_CB);
        carve_wide(c, Q, nb, wide_bound_plan(Q, nb, k), nullptr, nullptr);
        return c.size() + 256;
    }
    if (topk_use_wide_f32(Q, nb, k)) {
        carve_wide(c, Q, nb, wide_bound_plan(Q, nb, k), nullptr, nullptr);
        c.take<uint8_t>((size_t)nb * FW_NCH * 64);
        c.take<uint8_t>((size_t)Q->n * FW_NCH * 64);
        c.take<uint32_t>(1);
        c.take<uint64_t>((size_t)Q->n * topk_kcap(k));
        c.take<uint32_t>((size_t)Q->n * FW_CB);
        return c.size() + 256;
    }
    const int sp = topk_splits(Q->n, nb, topk_bm(k, Q->dtype, Q->dim, topk_side_words(Q->dtype, Q->metric, n_cand > 0)));
    if (sp > 1) c.take<uint64_t>((size_t)Q->n * sp * k);
    const BoundPlan bp = topk_bound_plan(Q, nb, k);
    if (bp.use) {
        const int64_t rows = std::min(Q->n, bp.chunk);
        c.take<uint32_t>((size_t)rows * bp.groups);
        c.take<uint32_t>(rows);
        c.take<int32_t>(rows);
        c.take<int32_t>(Q->n + 1);
        c.take<uint64_t>((size_t)rows * bp.cap);
    }
    return c.size() + 256;
}

onng_status launch_topk(const onng_vectors *Q, const onng_vectors *B, const int32_t *cand,
                        int64_t n_cand, int32_t k, int32_t exclude_self, int32_t *ids,
                        void *dists, void *ws, size_t ws_bytes, hipStream_t st) {
    if (!(Q->dtype == B->dtype && (Q->dtype == ONNG_U8 || Q->dtype == ONNG_F32))) {
        set_error("onng_topk: queries and base must both be u8 or both f32");
        return ONNG_ERR_UNSUPPORTED;
    }
    if (Q->dtype == ONNG_U8 && Q->metric != ONNG_L2SQ) {
        set_error("onng_topk: u8 data supports squared L2 only");
        return ONNG_ERR_UNSUPPORTED;
    }
    if (ws_bytes < topk_ws_size(Q, B, cand ? n_cand : 0, k)) {
        set_error("onng_topk: workspace too small");
        return ONNG_ERR_WORKSPACE;
    }
    if (Q->dim != B->dim || Q->dim > (Q->dtype == ONNG_U8 ? 512 : 256)) {
        set_error("onng_topk: dims differ, or above 512 (u8) / 256 (f32)");
        return ONNG_ERR_UNSUPPORTED;
    }
    const bool u8 = Q->dtype == ONNG_U8;
    const int64_t nb = cand ? n_cand : B->n;
    const bool wide = topk_use_wide(Q, nb, k);
    const bool wide_f32 = !wide && topk_use_wide_f32(Q, nb, k);
    Carver c(ws);
    void *qn = c.take<float>(Q->n);
    void *bn = c.take<float>(nb);
    const int sp = (wide || wide_f32) ? 1 : topk_splits(Q->n, nb, topk_bm(k, Q->dtype, Q->dim, topk_side_words(Q->dtype, Q->metric, cand != nullptr)));
    uint64_t *part = sp > 1 ? c.take<uint64_t>((size_t)Q->n * sp * k) : nullptr;
    const uint8_t *brows = static_cast<const uint8_t *>(B->data);
    uint8_t *gathered = cand && nb > 0 ? c.take<uint8_t>((size_t)nb * B->pitch_bytes) : nullptr;
    uint64_t *glist = wide ? c.take<uint64_t>((size_t)Q->n * topk_kcap(k)) : nullptr;
    uint64_t *gcand = wide ? c.take<uint64_t>((size_t)Q->n * WIDE_CB) : nullptr;
    uint8_t *fbh = nullptr, *fqh = nullptr;
    uint32_t *fymax = nullptr, *fcand = nullptr;
    uint64_t *flist = nullptr;
    if (wide_f32) {
        fbh = c.take<uint8_t>((size_t)nb * FW_NCH * 64);
        fqh = c.take<uint8_t>((size_t)Q->n * FW_NCH * 64);
        fymax = c.take<uint32_t>(1);
        flist = c.take<uint64_t>((size_t)Q->n * topk_kcap(k));
        fcand = c.take<uint32_t>((size_t)Q->n * FW_CB);
    }
    const BoundPlan bp = (wide || wide_f32) ? BoundPlan() : topk_bound_plan(Q, nb, k);
    uint32_t *mins = nullptr, *tau = nullptr;
    int32_t *cnt = nullptr, *redo = nullptr;
    uint64_t *bcand = nullptr;
    const WidePlan wp = wide || wide_f32 ? wide_bound_plan(Q, nb, k) : WidePlan();
    const WideBufs wb = carve_wide(c, Q, nb, wp, fbh, wide ? static_cast<void *>(gcand) : fqh);
    if (bp.use) {
        const int64_t rows = std::min(Q->n, bp.chunk);
        mins = c.take<uint32_t>((size_t)rows * bp.groups);
        tau = c.take<uint32_t>(rows);
        cnt = c.take<int32_t>(rows);
        redo = c.take<int32_t>(Q->n + 1);
        bcand = c.take<uint64_t>((size_t)rows * bp.cap);
    }
    auto norms = [&](const void *x, int64_t pitch, int64_t n, void *out) {
        if (n == 0) return;
        const dim3 grid((unsigned)((n + 3) / 4));
        if (u8)
            hipLaunchKernelGGL(norms_kernel<int32_t>, grid, dim3(256), 0, st,
                               static_cast<const uint8_t *>(x), pitch, n, Q->dim,
                               static_cast<int32_t *>(out));
        else
            hipLaunchKernelGGL(norms_kernel<float>, grid, dim3(256), 0, st,
                               static_cast<const uint8_t *>(x), pitch, n, Q->dim,
                               static_cast<float *>(out));
    };
    const bool query_norms = wide_f32 || u8 || Q->metric == ONNG_L2SQ;
    if (gathered) {
        const int64_t nn = query_norms ? Q->n : 0;
        const dim3 grid((unsigned)((nb + nn + 3) / 4));
        const uint8_t *q = static_cast<const uint8_t *>(Q->data);
        if (u8)
            hipLaunchKernelGGL(gather_norms_kernel<int32_t>, grid, dim3(256), 0, st, brows,
                               B->pitch_bytes, cand, nb, gathered, q, Q->pitch_bytes, nn, Q->dim,
                               static_cast<int32_t *>(qn));
        else
            hipLaunchKernelGGL(gather_norms_kernel<float>, grid, dim3(256), 0, st, brows,
                               B->pitch_bytes, cand, nb, gathered, q, Q->pitch_bytes, nn, Q->dim,
                               static_cast<float *>(qn));
        brows = gathered;
    }
    // Base norms: the wide kernels read them, and so does the list kernel where it
    // sweeps at least 32 tiles by itself (norms from the staged tiles are 12 % of its
    // time: 300,000 x 300 u8, k 10: 431 against 379 ms; a launch is 5 us).  The
    // others take them from the staged tiles, and cosine needs none.
    const bool list_norms = !wide && !wide_f32 && !bp.use && (u8 || Q->metric == ONNG_L2SQ) &&
                            (nb + BN - 1) / BN >= 32 * sp;
    if (wide || wide_f32 || list_norms) norms(brows, B->pitch_bytes, nb, bn);
    if (query_norms && !gathered) norms(Q->data, Q->pitch_bytes, Q->n, qn);
    ONNG_HIP(hipGetLastError());
    if (Q->n == 0) return ONNG_OK;

    TopkArgs a;
    a.q = static_cast<const uint8_t *>(Q->data);
    a.q_pitch = Q->pitch_bytes;
    a.nq = Q->n;
    a.b = brows;
    a.b_pitch = B->pitch_bytes;
    a.nb = nb;
    a.b_ids = cand;
    a.qn = qn;
    a.bn = wide || wide_f32 || list_norms ? bn : nullptr;
    a.dim = Q->dim;
    a.k = k;
    a.kcap = topk_kcap(k);
    a.cb = topk_cb(k);
    const int side_words = topk_side_words(Q->dtype, Q->metric, cand != nullptr);
    a.side_norms = Q->dtype == ONNG_U8 || Q->metric == ONNG_L2SQ;
    a.bm = topk_bm(k, Q->dtype, Q->dim, side_words);
    a.exclude_self = exclude_self;
    a.rotate = 0;   // set below once the split count is known
    a.only = nullptr;
    // the staged tile holds a row's components (zero-extended), not its padding
    a.lds_pitch = lds_pitch_for(Q->dtype, B->dim);
    a.out_ids = ids;
    a.out_d = dists;
    // the queries are the base rows: their converted copies serve both
    const bool same = !cand && Q->data == B->data && Q->n == B->n && Q->pitch_bytes == B->pitch_bytes;
    if (wide_f32) {
        a.splits = 1;
        a.tiles_per_split = (int)((nb + FW_BN - 1) / FW_BN);
        a.part = nullptr;
        a.rotate = same ? 1 : 0;
        if (wp.use) {
            const onng_status s = launch_wide_bound(a, Q, same, wp, wb, st);
            if (s != ONNG_OK) return s;
            a.only = wb.redo;   // rows that overflowed or fell short, if any
        }
        return launch_topk_wide_f32(a, Q, same, fqh, fbh, fymax, flist, fcand, st);
    }
    if (wide) {
        a.splits = 1;
        a.tiles_per_split = (int)((nb + BN - 1) / BN);
        a.part = nullptr;
        a.rotate = same ? 1 : 0;
        if (wp.use) {
            const onng_status s = launch_wide_bound(a, Q, same, wp, wb, st);
            if (s != ONNG_OK) return s;
            a.only = wb.redo;
        }
        return launch_topk_wide(a, nch_for(ONNG_U8, Q->dim), glist, gcand, st);
    }
    size_t lds = topk_lds_bytes(a.bm, a.kcap, a.cb, a.lds_pitch, side_words);
    if (lds > 160 * 1024) {
        set_error("onng_topk: k or dim too large for the on-chip tile");
        return ONNG_ERR_UNSUPPORTED;
    }
    if (bp.use) {
        BoundArgs ba;
        ba.t = a;
        ba.ns_log2 = bp.ns_log2;
        ba.group_tiles = bp.group_tiles;
        ba.quads = bp.quads;
        ba.groups = bp.groups;
        ba.mins = mins;
        ba.tau = tau;
        ba.cnt = cnt;
        ba.cand = bcand;
        ba.cap = bp.cap;
        auto fn_of = u8 ? topk_bound_fn_u8 : Q->metric == ONNG_L2SQ ? topk_bound_fn_l2 : topk_bound_fn_cosine;
        const int bm = bp.rw * 16;
        const int rank = k + (exclude_self ? 1 : 0);
        for (ba.row_first = 0; ba.row_first < Q->n; ba.row_first += bp.chunk) {
            const int64_t rows = std::min(bp.chunk, Q->n - ba.row_first);
            ba.t.nq = ba.row_first + rows;
            for (int m = 0; m < 2; m++) {
                const void *fn = fn_of(nch_for(Q->dtype, Q->dim), bp.rw, m == 0);
                ONNG_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bp.lds[m]));
                ba.t.tiles_per_split = bp.per_split[m];
                void *bargs[] = {&ba};
                ONNG_HIP(hipLaunchKernel(fn, dim3((unsigned)((rows + bm - 1) / bm), (unsigned)bp.splits[m]),
                                         dim3((unsigned)bound_threads(bp.rw)), bargs, bp.lds[m], st));
                // (u8: the bits of the largest distance, dim * 255^2, 25 of them at 512
                // components; f32 bounds need no more than 16 bits past the exponent's first)
                if (m == 0)
                    launch_bound_select(mins, rows, bp.groups, rank, bound_most(bp.cap, bp.ns_log2, nb),
                                        u8 ? 31 - __builtin_clz(Q->dim * 65025u) : 31, u8 ? 0 : 8, bp.cap, 1, 0, tau,
                                        cnt, ba.row_first == 0 ? redo : nullptr, st);
            }
            launch_bound_sort(u8, bcand, bp.cap, cnt, rows, k, false, ids, dists, redo, ba.row_first, st);
        }
        // rows that overflowed or fell short, if any
        a.only = redo;
    }
    const int nch = nch_for(Q->dtype, Q->dim);
    const void *fn;
    if (u8) fn = topk_fn_for<ONNG_U8, ONNG_L2SQ>(nch);
    else if (Q->metric == ONNG_L2SQ) fn = topk_fn_for<ONNG_F32, ONNG_L2SQ>(nch);
    else fn = topk_fn_for<ONNG_F32, ONNG_COSINE>(nch);
    ONNG_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int ntiles = (int)((nb + BN - 1) / BN);
    a.splits = sp;
    a.rotate = same && sp == 1 ? 1 : 0;
    a.tiles_per_split = (ntiles + sp - 1) / sp;
    a.part = part;
    dim3 grid((unsigned)((Q->n + a.bm - 1) / a.bm), (unsigned)sp),
        block((unsigned)(a.bm / 16 * 64));
    void *args[] = {&a};
    ONNG_HIP(hipLaunchKernel(fn, grid, block, args, lds, st));
    if (sp > 1) {
        const int wpb = 4;
        const size_t mlds = (size_t)wpb * (a.kcap + WAVE) * 8;
        const void *mf = u8 ? (const void *)merge_parts_kernel<true>
                            : (const void *)merge_parts_kernel<false>;
        ONNG_HIP(hipFuncSetAttribute(mf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)mlds));
        int64_t nq = Q->n;
        int splits = sp, kk = k, kcap = a.kcap;
        void *margs[] = {&part, &nq, &splits, &kk, &kcap, &ids, &dists, &a.only};
        ONNG_HIP(hipLaunchKernel(mf, dim3((unsigned)((Q->n + wpb - 1) / wpb)), dim3(wpb * WAVE),
                                 margs, mlds, st));
    }
    return ONNG_OK;
}

}  // namespace onng
