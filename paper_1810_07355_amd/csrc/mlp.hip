// Training kernels of the learned search range: a 2-layer perceptron
// F -> H (ReLU) -> T trained with a weighted mean squared error and Adam,
// all in f32.  Gradient sums over the batch use a fixed reduction order, so
// results are deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "pred_inputs.h"
#include "onng_internal.h"

namespace onng {

namespace {

// MLP_S samples per wave: hidden activations, outputs and, when target is
// given, dL/dy and dL/dh (the per-sample pieces of the gradient).  Lane j is
// hidden unit j, then lane s * 16 + t output t of sample s; every sum runs in
// index order in one lane.  The weights sit in LDS.  It is one chain of some
// 200 dependent multiply-adds, so what counts is that the batch fills the
// chip: 1024 samples are 256 waves.  (One thread per sample, its activations
// in scratch memory, 16 waves: 279 us at 1024 x (14 -> 64 -> 16); with four
// samples a wave 14.2 us, and 7.3 us since all inputs are requested at once.)
constexpr int MLP_S = 4;
constexpr int MLP_LDS_F = 32;   // widest input whose first layer is staged in LDS

__global__ void __launch_bounds__(64) mlp_sample_kernel(const float *X, int batch, int F,
                                                        const float *W1, const float *b1, int H,
                                                        const float *W2, const float *b2, int T,
                                                        const float *target, const float *w,
                                                        float *hid, float *Y, float *dy, float *dh,
                                                        float *lossp) {
    __shared__ float w1s[64 * MLP_LDS_F], w2s[16 * 65], xs[MLP_S * MLP_LDS_F], hs[MLP_S][64],
        gs[MLP_S][16], es[MLP_S][16], ws[MLP_S][16];
    const int lane = threadIdx.x;
    const int n0 = blockIdx.x * MLP_S;
    const int so = lane / 16, t = lane % 16;
    const int64_t n = n0 + so;
    const bool out = t < T && n < batch;
    // every input is requested before any is used: one trip to memory, where
    // loops of a load and its use took one each
    const float b1v = b1[min(lane, H - 1)], b2v = b2[min(t, T - 1)];
    const int64_t nt = out ? n * T + t : 0;
    const float tgt = target ? target[nt] : 0.0f;
    const float wt = target && w ? w[nt] : 1.0f;
    const bool staged = F <= MLP_LDS_F;
    const int nx = min(MLP_S, batch - n0) * F;
    float xr[MLP_S * MLP_LDS_F / 64], r2[16], r1[MLP_LDS_F / 2];
    if (staged) {
#pragma unroll
        for (int u = 0; u < MLP_S * MLP_LDS_F / 64; u++)
            xr[u] = X[(int64_t)n0 * F + min(lane + 64 * u, nx - 1)];
    }
#pragma unroll
    for (int u = 0; u < 16; u++) r2[u] = W2[min(lane + 64 * u, T * H - 1)];
    if (staged) {
        for (int i0 = 0; i0 < H * F; i0 += 64 * (MLP_LDS_F / 2)) {
#pragma unroll
            for (int u = 0; u < MLP_LDS_F / 2; u++) r1[u] = W1[min(i0 + lane + 64 * u, H * F - 1)];
#pragma unroll
            for (int u = 0; u < MLP_LDS_F / 2; u++) {
                const int i = i0 + lane + 64 * u;
                if (i < H * F) w1s[i] = r1[u];
            }
        }
#pragma unroll
        for (int u = 0; u < MLP_S * MLP_LDS_F / 64; u++)
            if (lane + 64 * u < nx) xs[lane + 64 * u] = xr[u];
    }
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int i = lane + 64 * u;
        // (64 hidden units: no division)
        if (i < T * H) w2s[H == 64 ? u * 65 + lane : i / H * 65 + i % H] = r2[u];
    }
    __syncthreads();
    float a[MLP_S];
#pragma unroll
    for (int s = 0; s < MLP_S; s++) a[s] = lane < H ? b1v : 0.0f;
    if (lane < H) {
        if (staged) {
            for (int i = 0; i < F; i++) {
                const float wi = w1s[lane * F + i];
#pragma unroll
                for (int s = 0; s < MLP_S; s++)
                    a[s] = fmaf(wi, xs[min(s, batch - 1 - n0) * F + i], a[s]);
            }
        } else {
            for (int i = 0; i < F; i++) {
                const float wi = W1[lane * F + i];
#pragma unroll
                for (int s = 0; s < MLP_S; s++)
                    a[s] = fmaf(wi, X[(int64_t)min(n0 + s, batch - 1) * F + i], a[s]);
            }
        }
    }
#pragma unroll
    for (int s = 0; s < MLP_S; s++) {
        const float h = fmaxf(a[s], 0.0f);
        hs[s][lane] = h;
        if (hid && lane < H && n0 + s < batch) hid[(int64_t)(n0 + s) * H + lane] = h;
    }
    __syncthreads();
    const float scale = 1.0f / ((float)batch * (float)T);
    if (out) {
        float y = b2v;
        for (int j = 0; j < H; j++) y = fmaf(w2s[t * 65 + j], hs[so][j], y);
        if (Y) Y[n * T + t] = y;
        if (target) {
            const float e = y - tgt;
            const float g = 2.0f * wt * e * scale;
            es[so][t] = e;
            ws[so][t] = wt;
            gs[so][t] = g;
            dy[n * T + t] = g;
        }
    }
    if (!target) return;
    __syncthreads();
    if (t == 0 && n < batch) {
        float l = 0.0f;
        for (int u = 0; u < T; u++) l += ws[so][u] * es[so][u] * es[so][u];
        lossp[n] = l * scale;
    }
    if (lane >= H) return;
#pragma unroll
    for (int s = 0; s < MLP_S; s++) {
        if (n0 + s >= batch) break;
        float d = 0.0f;
        for (int u = 0; u < T; u++) d = fmaf(w2s[u * 65 + lane], gs[s][u], d);
        dh[(int64_t)(n0 + s) * H + lane] = a[s] > 0.0f ? d : 0.0f;
    }
}

// Sums over the batch of the per-sample products, a lane a hidden unit (or
// output):
//   blocks [0, F)          gW1[j][i] = sum_n dh[n][j] x[n][i]
//   block F                gb1[j]    = sum_n dh[n][j]
//   blocks (F, F + T]      gW2[t][j] = sum_n dy[n][t] h[n][j]
//   block F + T + 1        gb2[t]    = sum_n dy[n][t]
//   block F + T + 2        loss      = sum_n lossp[n]
// The order of a sum is fixed: 256 partial sums (sample n in number n mod 256),
// added in pairs 128, 64, ..., 1 apart.  Wave v of 16 keeps the partial sums v,
// v + 16, ..., v + 240 in registers, so that it reads whole rows of dh or h; one
// block per parameter and a thread per partial sum read each row's line for 4
// bytes of it: 13.0 us at 1024 x (14 -> 64 -> 16), now 6.6 us.
// A wave may put G partial sums beside each other and take 64 / G units (blockIdx.y
// says which) over G times 256 samples at a time: see mlp_reduce_groups.
template <int G>
__global__ void __launch_bounds__(1024) mlp_reduce_kernel(const float *X, int batch, int F, int H,
                                                          int T, const float *hid, const float *dy,
                                                          const float *dh, const float *lossp,
                                                          float *gW1, float *gb1, float *gW2,
                                                          float *gb2, float *loss) {
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int p = blockIdx.x;
    // term(n) = row[n * pitch + lane] (* fac[n * fpitch] where fac)
    const float *row = dh, *fac = nullptr;
    int pitch = H, fpitch = 0, lanes = H, step = 1;
    float *dst = gb1;
    if (p < F) {
        fac = X + p; fpitch = F; dst = gW1 + p; step = F;
    } else if (p > F && p <= F + T) {
        row = hid; fac = dy + (p - F - 1); fpitch = T; dst = gW2 + (int64_t)(p - F - 1) * H;
    } else if (p == F + T + 1) {
        row = dy; pitch = T; lanes = T; dst = gb2;
    } else if (p == F + T + 2) {
        row = lossp; pitch = 1; lanes = 1; dst = loss;
    }
    // register u of lane group g: partial sum wave + 16 (u G + g)
    constexpr int W = 64 / G, R = 16 / G;
    if ((int)blockIdx.y * W >= lanes) return;
    const int col = min((int)blockIdx.y * W + lane % W, lanes - 1);
    const int first = G == 1 ? wave : wave + 16 * (lane / W);
    float s[R];
#pragma unroll
    for (int u = 0; u < R; u++) s[u] = 0.0f;
    for (int n0 = first; n0 < batch; n0 += 256 * G) {
        float v[16], f[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int64_t n = min(n0 + 256 * (i / R) + 16 * G * (i % R), batch - 1);
            v[i] = row[n * pitch + col];
            f[i] = fac ? fac[n * fpitch] : 1.0f;
        }
#pragma unroll
        for (int i = 0; i < 16; i++)
            if (n0 + 256 * (i / R) + 16 * G * (i % R) < batch) s[i % R] = fmaf(v[i], f[i], s[i % R]);
    }
#pragma unroll
    for (int m = R / 2; m >= 1; m >>= 1)
#pragma unroll
        for (int u = 0; u < m; u++) s[u] += s[u + m];
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) s[0] += __shfl_down(s[0], m * W);
    red[wave][lane] = s[0];
    __syncthreads();
    const int unit = blockIdx.y * W + lane;
    if (wave != 0 || lane >= W || unit >= lanes) return;
    float r[16];
#pragma unroll
    for (int v = 0; v < 16; v++) r[v] = red[v][lane];
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1)
#pragma unroll
        for (int v = 0; v < m; v++) r[v] += r[v + m];
    dst[unit * step] = r[0];
}

__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float mi = b1 * m[i] + (1.0f - b1) * g[i];
    float vi = b2 * v[i] + (1.0f - b2) * g[i] * g[i];
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// the transform the fused predictor of the search applies before z-scoring
__global__ void feature_transform_kernel(const float *raw, int64_t n, int metric, float *out) {
    int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const float *f = raw + r * ONNG_NFEAT;
    float *x = out + r * ONNG_NFEAT;
    for (int t = 0; t < ONNG_NFEAT; t++) x[t] = feature_input(t, f[t], f[0], metric);
}

// Per-column mean and standard deviation of x [n][cols] (weights w [n][cols]
// or all ones): one block per column, sums in double, the deviations in a
// second pass over the column.  A standard deviation below 1e-6 becomes 1.
__global__ void column_stats_kernel(const float *x, const float *w, int64_t n, int cols,
                                    float *mean, float *stdv) {
    __shared__ double red[2][256];
    const int c = blockIdx.x;
    double sw = 0.0, sx = 0.0;
    for (int64_t r = threadIdx.x; r < n; r += blockDim.x) {
        const double wi = w ? (double)w[r * cols + c] : 1.0;
        sw += wi;
        sx += wi * (double)x[r * cols + c];
    }
    red[0][threadIdx.x] = sw;
    red[1][threadIdx.x] = sx;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) {
            red[0][threadIdx.x] += red[0][threadIdx.x + h];
            red[1][threadIdx.x] += red[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    const double tot = red[0][0] > 1e-12 ? red[0][0] : 1e-12;
    const double mu = red[1][0] / tot;
    __syncthreads();
    double sv = 0.0;
    for (int64_t r = threadIdx.x; r < n; r += blockDim.x) {
        const double wi = w ? (double)w[r * cols + c] : 1.0;
        const double d = (double)x[r * cols + c] - mu;
        sv += wi * d * d;
    }
    red[0][threadIdx.x] = sv;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) red[0][threadIdx.x] += red[0][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double sd = sqrt(red[0][0] / tot);
        mean[c] = (float)mu;
        stdv[c] = sd < 1e-6 ? 1.0f : (float)sd;
    }
}

__global__ void standardize_kernel(const float *x, int64_t n, int cols, const float *mean,
                                   const float *stdv, float *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * cols) return;
    const int c = (int)(i % cols);
    out[i] = (x[i] - mean[c]) / stdv[c];
}

// W2 [T][H] and b2 [T] of a network trained on targets (y - shift) / scale:
// the same network on the targets themselves.
__global__ void fold_output_kernel(float *w2, float *b2, int T, int H, const float *scale,
                                   const float *shift) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < T * H) w2[i] *= scale[i / H];
    if (i < T) b2[i] = b2[i] * scale[i] + shift[i];
}

}  // namespace

onng_status column_stats_launch(const float *x, const float *w, int64_t n, int32_t cols,
                                float *mean, float *stdv, hipStream_t st) {
    if (cols == 0) return ONNG_OK;
    hipLaunchKernelGGL(column_stats_kernel, dim3((unsigned)cols), dim3(256), 0, st, x, w, n, cols,
                       mean, stdv);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

onng_status standardize_launch(const float *x, int64_t n, int32_t cols, const float *mean,
                               const float *stdv, float *out, hipStream_t st) {
    if (n == 0 || cols == 0) return ONNG_OK;
    hipLaunchKernelGGL(standardize_kernel, dim3((unsigned)((n * cols + 255) / 256)), dim3(256), 0,
                       st, x, n, cols, mean, stdv, out);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

onng_status fold_output_launch(float *w2, float *b2, int32_t T, int32_t H, const float *scale,
                               const float *shift, hipStream_t st) {
    if (T == 0) return ONNG_OK;
    const int m = T * H > T ? T * H : T;
    hipLaunchKernelGGL(fold_output_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, w2,
                       b2, T, H, scale, shift);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

size_t mlp_backward_ws(int32_t batch, int32_t H, int32_t T) {
    Carver c(nullptr);
    c.take<float>((size_t)batch * H);   // hidden
    c.take<float>((size_t)batch * T);   // dy
    c.take<float>((size_t)batch * H);   // dh
    c.take<float>((size_t)batch);       // per-sample loss
    return c.size() + 256;
}

onng_status mlp_forward_launch(const float *X, int32_t batch, int32_t F, const float *W1,
                               const float *b1, int32_t H, const float *W2, const float *b2,
                               int32_t T, float *hidden, float *Y, hipStream_t st) {
    if (batch == 0) return ONNG_OK;
    hipLaunchKernelGGL(mlp_sample_kernel, dim3((batch + MLP_S - 1) / MLP_S), dim3(64), 0, st, X, batch,
                       F, W1, b1, H, W2, b2, T, nullptr, nullptr, hidden, Y, nullptr, nullptr,
                       nullptr);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

// Partial sums beside each other in a wave of the gradient sums.  A wave takes 256 G
// samples at a time, so up to 2048 samples one time or a few; from there on the few
// blocks of whole rows leave the chip idle, and the units are split as far as the
// blocks stay within one per compute unit.  Backward at 100,000 samples, us, with
// G = 1, so, and with a block per parameter: 14 -> 16 -> 2: 539, 245, 214; 5 -> 33 ->
// 2: 541, 268, 257; 14 -> 64 -> 16: 555, 303, 1761 (at 20,000: 114, 50, 73; 117, 57,
// 91; 120, 67, 517).
static int mlp_reduce_groups(int32_t batch, int32_t F, int32_t H, int32_t T) {
    const int lanes = std::max(H, T);
    int G = 1;
    if (batch >= 2048)
        while (G < 16 && (int64_t)(F + T + 3) * ((lanes + 32 / G - 1) / (32 / G)) <= device_cu_count()) G *= 2;
    return G;
}

onng_status mlp_backward_launch(const float *X, const float *target, const float *w,
                                int32_t batch, int32_t F, const float *W1, const float *b1,
                                int32_t H, const float *W2, const float *b2, int32_t T,
                                float *gW1, float *gb1, float *gW2, float *gb2, float *loss,
                                void *ws, hipStream_t st) {
    Carver c(ws);
    float *hid = c.take<float>((size_t)batch * H);
    float *dy = c.take<float>((size_t)batch * T);
    float *dh = c.take<float>((size_t)batch * H);
    float *lp = c.take<float>((size_t)batch);
    hipLaunchKernelGGL(mlp_sample_kernel, dim3((batch + MLP_S - 1) / MLP_S), dim3(64), 0, st, X, batch,
                       F, W1, b1, H, W2, b2, T, target, w, hid, nullptr, dy, dh, lp);
    const int G = mlp_reduce_groups(batch, F, H, T);
    auto reduce = G == 16 ? mlp_reduce_kernel<16> : G == 8 ? mlp_reduce_kernel<8> : G == 4 ? mlp_reduce_kernel<4>
                  : G == 2 ? mlp_reduce_kernel<2> : mlp_reduce_kernel<1>;
    const int W = 64 / G;
    hipLaunchKernelGGL(reduce, dim3(F + T + 3, (std::max(H, T) + W - 1) / W), dim3(1024), 0, st, X, batch, F,
                       H, T, hid, dy, dh, lp, gW1, gb1, gW2, gb2, loss);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

onng_status adam_launch(float *p, const float *g, float *m, float *v, int64_t n, float lr,
                        float b1, float b2, float eps, int32_t t, hipStream_t st) {
    if (n == 0) return ONNG_OK;
    float c1 = (float)(1.0 - std::pow((double)b1, (double)t));
    float c2 = (float)(1.0 - std::pow((double)b2, (double)t));
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, g, m,
                       v, n, lr, b1, b2, eps, c1, c2);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

onng_status feature_transform_launch(const float *raw, int64_t n, int32_t metric, float *out,
                                     hipStream_t st) {
    if (n == 0) return ONNG_OK;
    hipLaunchKernelGGL(feature_transform_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       st, raw, n, metric, out);
    ONNG_HIP(hipGetLastError());
    return ONNG_OK;
}

}  // namespace onng
