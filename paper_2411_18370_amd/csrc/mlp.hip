// Detection-probability surrogate: MLP 6 -> 256 -> 256 -> 256 -> 1, GELU
// hidden activations, sigmoid output, binary cross-entropy, Adam -- trained
// and run on the GPU.  It estimates p_det of Sec. V (Eqs. pdet_abstract and
// sampling) from injection parameters.
//
// The two 256 x 256 layers (forward, input-gradient and weight-gradient
// products) run on the matrix cores: v_mfma_f32_16x16x32_bf16, BF16 operands,
// FP32 accumulation.  Master weights, biases, Adam moments, pre-activations and
// gradients are FP32; activations and the 256 x 256 weights feed the MFMAs in
// BF16.  The 6-wide input layer and the 1-wide output layer run on the VALU.
//
// Parameter vector (flat FP32): W1 [256][6], b1 [256], W2 [256][256], b2,
// W3 [256][256], b3, W4 [256], b4 -- 133,633 values; Z_l = A_{l-1} W_l^T + b_l.
//
// A query is one launch over all rows and a training step two: one over rows
// of the batch (forward, loss and the chain of dZ, activations handed from
// layer to layer through LDS), one over parameters (weight-gradient products
// over the batch in up to 8 slices, column sums in chunks of 64 rows, Adam and
// the BF16 copies).  Every reduction is deterministic: k in steps of 32 within
// a slice, slices and chunks in order.
#include <algorithm>
#include <type_traits>

#include "ft_internal.h"

namespace ft {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int H = 256;
constexpr int ACT_LD = H + 8;  // LDS row of activations: rows 4 banks apart

// Phi(x) 2 = 1 + erf(x / sqrt 2), shared by the activation and its derivative.
__device__ __forceinline__ float erf1(float x) { return 1.0f + erff(x * 0.70710678118654752f); }
__device__ __forceinline__ float gelu(float x, float e1) { return 0.5f * x * e1; }
__device__ __forceinline__ float gelu_grad(float x, float e1)
{
    const float cdf = 0.5f * e1;
    const float pdf = expf(-0.5f * x * x) * 0.39894228040143268f;
    return cdf + x * pdf;
}

// Standardised features of sample idx(b): (log amp, cos iota, psi, sin delta,
// alpha, f) -> (g - shift)/scale.
__device__ __forceinline__ float feature(const float *raw, int64_t s, int i, const MlpConst &c)
{
    float g = raw[s * 6 + i];
    if (i == 0) g = logf(g);
    return (g - c.shift[i]) / c.scale[i];
}

__device__ __forceinline__ int64_t sample_index(int64_t b, const MlpConst &c)
{
    return c.perm_a == 0 ? c.base + b : (int64_t)((c.perm_a * (uint64_t)(c.base + b) + c.perm_c) % (uint64_t)c.n_total);
}

// Position of W(n, k) (column n of the product, k summed) in a BF16 weight copy:
// 16-column by 32-k blocks in the order of the MFMA's B operand, so a wave's
// load of a block is 1 KB in a row.
__device__ __forceinline__ int frag_pos(int n, int k)
{
    return ((n >> 4) * (H / 32) + (k >> 5)) * 512 + (((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// Rows of a batch through the network, 16 RB of them a workgroup: wave w owns
// columns 32 w .. 32 w + 31 of every layer, holds its share of a weight matrix
// in 64 registers a lane and reads the layer's input rows from LDS.  TRAIN adds
// loss, dlogit and the chain dZ3, dZ2, dZ1; Z stays in registers (the products
// of the backward layers come out in the lanes that hold the forward ones),
// and what the parameter gradients need is written transposed, [column][row],
// so that they read it along the batch.  Padding rows (b >= bsz) have zero
// features and zero dZ.
//
// Without TRAIN a workgroup keeps both matrices in registers and walks over
// tiles: nothing but features is read, and the bound is the VALU's erf
// (measured at 200,000 rows: PREDICT_FIG).  A training step of 2048 rows has
// 128 workgroups: bound by the latency of the five layers in turn and the
// weights from L2 (STEP_FIG).
template <int RB, bool TRAIN>
__global__ __launch_bounds__(512) void mlp_rows_kernel(const float *raw, const float *labels, MlpBufs m, MlpConst c,
                                                       int bsz, int n_tiles, float inv_n, float *prob)
{
    constexpr int R = 16 * RB;
    __shared__ __bf16 act[2][R][ACT_LD];
    __shared__ float xs[R][6], ys[R], dl[R];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int n0 = 32 * wave + lr;  // the lane's columns: n0, n0 + 16
    const int64_t ld = m.ld;
    const float *th = m.theta;

    bf16x8 wa[2][8], wb[2][8];
    auto load_w = [&](const __bf16 *w, bf16x8 (&f)[2][8]) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int t = 0; t < 8; ++t) f[j][t] = *(const bf16x8 *)(w + ((2 * wave + j) * 8 + t) * 512 + lane * 8);
    };
    f32x4 acc[RB][2];
    auto product = [&](const __bf16 (*in)[ACT_LD], const bf16x8 (&f)[2][8]) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 8; ++t) {
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const bf16x8 a = *(const bf16x8 *)&in[16 * i + lr][32 * t + 8 * lg];
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, f[j][t], acc[i][j], 0, 0, 0);
            }
        }
    };
    // The lane's values of a layer: column n0 + 16 j, rows 16 i + 4 lg + r.
    f32x4 z[3][RB][2], e1[3][RB][2];
    auto activate = [&](int l, __bf16 (*out)[ACT_LD], __bf16 *glob, int b0) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bf16x4 a;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * i + 4 * lg + r;
                    e1[l][i][j][r] = erf1(z[l][i][j][r]);
                    a[r] = (__bf16)gelu(z[l][i][j][r], e1[l][i][j][r]);
                    if (l == 0 && b0 + row >= bsz) a[r] = (__bf16)0.f;
                    out[row][n0 + 16 * j] = a[r];
                }
                if (TRAIN) *(bf16x4 *)(glob + (n0 + 16 * j) * ld + b0 + 16 * i + 4 * lg) = a;
            }
    };
    auto bias_add = [&](int l, const float *bias) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float bj = bias[n0 + 16 * j];
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) z[l][i][j][r] = acc[i][j][r] + bj;
        }
    };
    // dZ of a layer from d (acc): dZ = d gelu'(Z), to LDS and, transposed, to memory
    auto derive = [&](int l, __bf16 (*out)[ACT_LD], float *gf, __bf16 *gb, int b0) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4 d;
                bf16x4 db;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * i + 4 * lg + r;
                    d[r] = acc[i][j][r] * gelu_grad(z[l][i][j][r], e1[l][i][j][r]);
                    if (l == 2 && b0 + row >= bsz) d[r] = 0.f;
                    db[r] = (__bf16)d[r];
                    if (out) out[row][n0 + 16 * j] = db[r];
                }
                const int64_t o = (n0 + 16 * j) * ld + b0 + 16 * i + 4 * lg;
                *(f32x4 *)(gf + o) = d;
                if (gb) *(bf16x4 *)(gb + o) = db;
            }
    };

    load_w(m.w2b, wa);
    load_w(m.w3b, wb);
    float w1[2][6], b1[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        b1[j] = th[6 * H + n0 + 16 * j];
#pragma unroll
        for (int q = 0; q < 6; ++q) w1[j][q] = th[(n0 + 16 * j) * 6 + q];
    }
    int tile = blockIdx.x;  // below n_tiles
    do {
        const int b0 = tile * R;
        __syncthreads();  // the last tile's rows are no longer read
        for (int q = tid; q < 8 * R; q += 512) {
            const int row = q >> 3, i = q & 7, b = b0 + row;
            const int64_t s = b < bsz ? sample_index(b, c) : 0;
            if (i < 6) {
                const float x = b < bsz ? feature(raw, s, i, c) : 0.f;
                xs[row][i] = x;
                if (TRAIN) m.x[i * ld + b] = x;
            } else if (TRAIN && i == 6) {
                ys[row] = b < bsz ? labels[s] : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * i + 4 * lg + r;
                float x[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) x[q] = xs[row][q];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    float v = b1[j];
#pragma unroll
                    for (int q = 0; q < 6; ++q) v += w1[j][q] * x[q];
                    z[0][i][j][r] = b0 + row < bsz ? v : 0.f;
                }
            }
        activate(0, act[0], m.a1, b0);
        __syncthreads();
        product(act[0], wa);
        if (TRAIN) load_w(m.w3t, wa);
        bias_add(1, th + MLP_OFF_W2 + H * H);
        activate(1, act[1], m.a2, b0);
        __syncthreads();
        product(act[1], wb);
        if (TRAIN) load_w(m.w2t, wb);
        bias_add(2, th + MLP_OFF_W3 + H * H);
        activate(2, act[0], m.a3, b0);
        __syncthreads();
        // output layer and sigmoid, a row a wave
        for (int row = wave; row < R; row += 8) {
            const int b = b0 + row;
            if (b >= bsz) {
                if (TRAIN && lane == 0) dl[row] = 0.f;
                continue;
            }
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < H; i += 64) s += th[MLP_OFF_W4 + i + lane] * (float)act[0][row][i + lane];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            const float zo = s + th[MLP_OFF_W4 + H];
            const float p = 1.f / (1.f + expf(-zo));
            if (lane != 0) continue;
            if (!TRAIN) {
                prob[b] = p;
                continue;
            }
            const float y = ys[row], d = (p - y) * inv_n;
            dl[row] = d;
            m.dlogit[b] = d;
            m.lossv[b] = fmaxf(zo, 0.f) - zo * y + log1pf(expf(-fabsf(zo)));
        }
        if (!TRAIN) continue;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float w4 = th[MLP_OFF_W4 + n0 + 16 * j];
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = dl[16 * i + 4 * lg + r] * w4;
        }
        derive(2, act[1], m.dz3, m.dz3b, b0);
        __syncthreads();
        product(act[1], wa);
        derive(1, act[0], m.dz2, m.dz2b, b0);
        __syncthreads();
        product(act[0], wb);
        derive(0, nullptr, m.dz1, nullptr, b0);
    } while (!TRAIN && (tile += gridDim.x) < n_tiles);
}

// Adam (Kingma and Ba 2015, bias-corrected); off: the gradient is stored instead.
struct AdamArgs {
    bool on;
    float lr, b1, b2, eps, c1, c2;
};

// Finishes parameter i, whose gradient is gi; returns its new value.
__device__ __forceinline__ float adam_step(const MlpBufs &m, const AdamArgs &ad, int i, float gi)
{
    if (!ad.on) {
        m.grad[i] = gi;
        return 0.f;
    }
    const float mi = ad.b1 * m.m[i] + (1.f - ad.b1) * gi;
    const float vi = ad.b2 * m.v[i] + (1.f - ad.b2) * gi * gi;
    m.m[i] = mi;
    m.v[i] = vi;
    const float t = m.theta[i] - ad.lr * (mi / ad.c1) / (sqrtf(vi / ad.c2) + ad.eps);
    m.theta[i] = t;
    return t;
}

// Every parameter's gradient and update.  Workgroups by blockIdx:
//   [0, 128)    32 x 32 tiles of W2 and W3: wave z forms slice z of the product
//               over the batch, the slices are added in order
//   [128, 192)  16 columns of one section of column sums (W1 and b1; b2; b3; W4
//               and b4): a thread sums a chunk of MLP_RED_ROWS rows, rows
//               b0 + w, b0 + w + 4, ... for w = 0..3 and the four in order, then
//               the chunks are added in order
//   192         the batch's mean loss
constexpr int UPD_W = 128, UPD_C = 64;

__global__ __launch_bounds__(512) void mlp_update_kernel(MlpBufs m, int bsz, int m_pad, int n_slices, int k_slice,
                                                         float inv_n, AdamArgs ad)
{
    __shared__ float red[8 * 32 * 33];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t ld = m.ld;
    if (blockIdx.x < UPD_W) {
        const bool w3 = blockIdx.x >= UPD_W / 2;
        const int o0 = (blockIdx.x >> 3 & 7) * 32, i0 = (blockIdx.x & 7) * 32;
        const __bf16 *A = (w3 ? m.dz3b : m.dz2b) + (o0 + (lane & 15)) * ld + 8 * (lane >> 4);
        const __bf16 *B = (w3 ? m.a2 : m.a1) + (i0 + (lane & 15)) * ld + 8 * (lane >> 4);
        f32x4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (wave < n_slices) {
            const int k1 = min(m_pad, (wave + 1) * k_slice);
            int k = wave * k_slice;
            auto steps = [&](auto n_c) {  // n steps of 32, loads ahead of the products
                constexpr int n = decltype(n_c)::value;
                bf16x8 a[n][2], b[n][2];
#pragma unroll
                for (int t = 0; t < n; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        a[t][i] = *(const bf16x8 *)(A + 16 * i * ld + k + 32 * t);
                        b[t][i] = *(const bf16x8 *)(B + 16 * i * ld + k + 32 * t);
                    }
#pragma unroll
                for (int t = 0; t < n; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][i], b[t][j], acc[i][j], 0, 0, 0);
                k += 32 * n;
            };
            while (k + 256 <= k1) steps(std::integral_constant<int, 8>());
            while (k < k1) steps(std::integral_constant<int, 1>());
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        red[(wave * 32 + 16 * i + 4 * (lane >> 4) + r) * 33 + 16 * j + (lane & 15)] = acc[i][j][r];
        }
        __syncthreads();
        __bf16 *wf = w3 ? m.w3b : m.w2b, *wt = w3 ? m.w3t : m.w2t;
        for (int q = tid; q < 1024; q += 512) {
            const int o = q >> 5, i = q & 31;
            float gi = 0.f;
            for (int z = 0; z < n_slices; ++z) gi += red[(z * 32 + o) * 33 + i];
            const float t = adam_step(m, ad, (w3 ? MLP_OFF_W3 : MLP_OFF_W2) + (o0 + o) * H + i0 + i, gi);
            if (!ad.on) continue;
            wf[frag_pos(o0 + o, i0 + i)] = (__bf16)t;
            wt[frag_pos(i0 + i, o0 + o)] = (__bf16)t;
        }
    } else if (blockIdx.x < UPD_W + UPD_C) {
        const int sec = (blockIdx.x - UPD_W) >> 4, j0 = ((blockIdx.x - UPD_W) & 15) * 16;
        const int col = tid & 15, j = j0 + col;  // chunk tid / 16 of each 32
        const int n_ent = sec == 0 ? 7 : sec == 3 ? 2 : 1;
        const int n_chunks = (bsz + MLP_RED_ROWS - 1) / MLP_RED_ROWS;
        const float *dz = (sec == 0 ? m.dz1 : sec == 1 ? m.dz2 : m.dz3) + j * ld;
        const __bf16 *a3 = m.a3 + j * ld;
        float sum = 0.f;  // thread 16 e + col: entry e of column j
        for (int c0 = 0; c0 < n_chunks; c0 += 32) {
            const int chunk = c0 + (tid >> 4);
            if (chunk < n_chunks) {
                const int b0 = chunk * MLP_RED_ROWS, nb = min(MLP_RED_ROWS, bsz - b0);
                float t[7][4];
#pragma unroll
                for (int e = 0; e < 7; ++e)
#pragma unroll
                    for (int w = 0; w < 4; ++w) t[e][w] = 0.f;
                // the batch is padded to whole chunks: four rows at a time
#pragma unroll 4
                for (int b = 0; b < nb; b += 4) {
                    if (sec < 3) {
                        const f32x4 d = *(const f32x4 *)(dz + b0 + b);
                        f32x4 x[6];
                        if (sec == 0)
#pragma unroll
                            for (int e = 0; e < 6; ++e) x[e] = *(const f32x4 *)(m.x + e * ld + b0 + b);
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            if (b + w >= nb) continue;
                            if (sec == 0) {
#pragma unroll
                                for (int e = 0; e < 6; ++e) t[e][w] += d[w] * x[e][w];
                                t[6][w] += d[w];
                            } else {
                                t[0][w] += d[w];
                            }
                        }
                    } else {
                        const f32x4 d = *(const f32x4 *)(m.dlogit + b0 + b);
                        const bf16x4 a = *(const bf16x4 *)(a3 + b0 + b);
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            if (b + w >= nb) continue;
                            t[0][w] += d[w] * (float)a[w];
                            t[1][w] += d[w];
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (e < n_ent) red[(tid >> 4) * 112 + 16 * e + col] = ((t[e][0] + t[e][1]) + t[e][2]) + t[e][3];
            }
            __syncthreads();
            if (tid < 16 * n_ent)
                for (int q = 0; q < min(32, n_chunks - c0); ++q) sum += red[q * 112 + tid];
            __syncthreads();
        }
        if (tid < 16 * n_ent) {
            const int e = tid >> 4;
            const int i = sec == 0 ? (e < 6 ? 6 * j + e : 6 * H + j)
                          : sec == 1 ? MLP_OFF_W2 + H * H + j
                          : sec == 2 ? MLP_OFF_W3 + H * H + j
                                     : MLP_OFF_W4 + (e == 0 ? j : H);
            if (!(sec == 3 && e == 1 && j != 0)) adam_step(m, ad, i, sum);
        }
    } else {
        if (tid < 256) {
            float t = 0.f;
            for (int b = tid; b < bsz; b += 256) t += m.lossv[b];
            red[tid] = t;
        }
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) red[tid] += red[tid + w];
            __syncthreads();
        }
        if (tid == 0) *m.loss += red[0] * inv_n;
    }
}

// BF16 copies of a 256 x 256 weight matrix, as it stands and transposed.
__global__ void to_bf16_kernel(const float *src, __bf16 *dst, __bf16 *dst_t)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= H * H) return;
    dst[frag_pos(r / H, r % H)] = (__bf16)src[r];
    dst_t[frag_pos(r % H, r / H)] = (__bf16)src[r];
}

// First inadmissible value: bad[0] = least 2 i (amplitude of sample i not > 0)
// or 2 i + 1 (another input not finite), bad[1] = 0 where a label lies outside
// [0, 1]; both stay at their all-ones start otherwise.
__global__ __launch_bounds__(256) void mlp_check_kernel(const float *raw, const float *y, int64_t n, uint64_t *bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t key = ~0ull;
    bool label = false;
    if (i < n) {
        bool fin = true;
        for (int j = 0; j < 6; ++j) fin = fin && __builtin_isfinite(raw[i * 6 + j]);
        if (!(raw[i * 6] > 0.0f)) key = 2 * (uint64_t)i;
        else if (!fin) key = 2 * (uint64_t)i + 1;
        label = y && !(y[i] >= 0.0f && y[i] <= 1.0f);
    }
    if (key != ~0ull) atomicMin((unsigned long long *)bad, (unsigned long long)key);
    if (label) bad[1] = 0;
}

unsigned blocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t mlp_refresh_bf16(const MlpBufs &m, hipStream_t s)
{
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks(H * H, 256)), dim3(256), 0, s,
                       m.theta + MLP_OFF_W2, m.w2b, m.w2t);
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks(H * H, 256)), dim3(256), 0, s,
                       m.theta + MLP_OFF_W3, m.w3b, m.w3t);
    return hipGetLastError();
}

hipError_t mlp_check(const float *raw, const float *y, int64_t n, uint64_t *bad, hipStream_t s)
{
    hipLaunchKernelGGL(mlp_check_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, raw, y, n, bad);
    return hipGetLastError();
}

hipError_t mlp_predict(const MlpBufs &m, const float *raw, const MlpConst &c, int n, float *prob, hipStream_t s)
{
    // one tile of 16 rows a workgroup while that is one round of the 256 CUs
    if (n <= 16 * 256) {
        const int tiles = (n + 15) / 16;
        hipLaunchKernelGGL((mlp_rows_kernel<1, false>), dim3(tiles), dim3(512), 0, s, raw, nullptr, m, c, n, tiles, 0.f, prob);
    } else {
        const int tiles = (int)(((int64_t)n + 31) / 32);
        hipLaunchKernelGGL((mlp_rows_kernel<2, false>), dim3(std::min(tiles, 256)), dim3(512), 0, s, raw, nullptr, m, c, n,
                           tiles, 0.f, prob);
    }
    return hipGetLastError();
}

// Loss and gradient of samples [c.base, c.base + bsz): the gradient into
// m.grad or, with adam, one Adam step t; the batch's mean loss is added to *m.loss.
hipError_t mlp_step(const MlpBufs &m, const float *raw, const float *labels, const MlpConst &c, int bsz,
                    const MlpAdamStep *adam, hipStream_t s)
{
    const int m_pad = (bsz + 63) / 64 * 64;
    const float inv_n = 1.f / (float)bsz;
    hipLaunchKernelGGL((mlp_rows_kernel<1, true>), dim3(m_pad / 16), dim3(512), 0, s, raw, labels, m, c, bsz, m_pad / 16,
                       inv_n, nullptr);
    // the weight-gradient products sum over the batch in slices of >= 256 rows
    const int n_sl = std::max(1, std::min(MLP_MAX_SLICES, m_pad / 256));
    const int k_sl = (m_pad / n_sl + 31) / 32 * 32;
    AdamArgs ad{false, 0.f, 0.9f, 0.999f, 1e-8f, 1.f, 1.f};
    if (adam) {
        ad.on = true;
        ad.lr = adam->lr;
        ad.c1 = 1.f - powf(ad.b1, (float)adam->t);
        ad.c2 = 1.f - powf(ad.b2, (float)adam->t);
    }
    hipLaunchKernelGGL(mlp_update_kernel, dim3(UPD_W + UPD_C + 1), dim3(512), 0, s, m, bsz, m_pad, n_sl, k_sl, inv_n, ad);
    return hipGetLastError();
}

}  // namespace ft
