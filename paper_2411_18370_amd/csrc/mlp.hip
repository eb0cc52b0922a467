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

// 1 + erf(x / sqrt 2), shared by the activation and its derivative.
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
__device__ __forceinline__ float feature(float g, int i, const MlpConst &c)
{
    if (i == 0) g = logf(g);
    return (g - c.shift[i]) / c.scale[i];
}

// (perm_a b + start) mod n_total, start the value at b = 0.  The
// quotient from FP64 is at most one off.
__device__ __forceinline__ int64_t sample_index(int64_t b, const MlpConst &c)
{
    if (c.perm_a == 0) return c.base + b;
    const uint64_t v = c.perm_a * (uint64_t)b + c.start, n = (uint64_t)c.n_total;
    int64_t r = (int64_t)(v - (uint64_t)((double)v * c.inv_total) * n);
    if (r < 0) r += n;
    if (r >= (int64_t)n) r -= n;
    return r;
}

// Position of W(n, k) (column n of the product, k summed) in a BF16 weight copy:
// 16-column by 32-k blocks in the order of the MFMA's B operand, so a wave's
// load of a block is 1 KB in a row.
__device__ __forceinline__ int frag_pos(int n, int k)
{
    return ((n >> 4) * (H / 32) + (k >> 5)) * 512 + (((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// What a step's rows leave for the parameters, by unit n and row b of the batch
// (ld rows held).  unit_frag: BF16 operands of the products over the batch, in
// the blocks of frag_pos with k = b (a wave's load of [unit][row] rows took one
// lane a clock, four times as long).  unit_col: FP32 dZ and A3 for the column
// sums, 8 units by 4 rows in a row.
__device__ __forceinline__ int64_t unit_frag(int n, int b, int64_t ld)
{
    return ((n >> 4) * (ld >> 5) + (b >> 5)) * 512 + (((b >> 3) & 3) * 16 + (n & 15)) * 8 + (b & 7);
}
__device__ __forceinline__ int64_t unit_col(int n, int b, int64_t ld)
{
    return ((n >> 3) * (ld >> 2) + (b >> 2)) * 32 + (n & 7) * 4 + (b & 3);
}

// Threads of a workgroup of rows: 8 waves of two 16-column blocks (R = 8) or 16
// waves of one.
constexpr int row_threads(int r) { return 64 * r; }

// Rows of a batch through the network, R of them a workgroup (8 or 16): a
// wave owns 32 or 16 columns of every layer, holds its share of two weight
// matrices in registers and reads the layer's input rows from LDS.  TRAIN adds
// loss, dlogit and the chain dZ3, dZ2, dZ1; Z stays in registers (the products
// of the backward layers come out in the lanes that hold the forward ones), and
// what the parameter gradients need is written in the order they read it.  Padding rows (b >= bsz) have zero
// features and zero dZ.
//
// R = 8 fills the 16 rows of a product with each row twice; of the duplicate
// results the lower half of the lanes keeps the first 16 columns' and the upper
// half the second's, so the VALU work is halved all the same.
//
// Without TRAIN a workgroup keeps both matrices and walks over tiles: nothing
// but features is read, and the bound is the VALU's erf (two branches each, so a
// lane's run one after the other and take waves to overlap; 200,000 rows: 233 us
// with the VALU 81% busy, 1200 us as four launches per 8192 rows).  A training
// step's workgroups are bound by the latency of five layers in turn, the first
// behind the weights' way from L2 (2048 rows: 17 us, VALU 27% busy; 59 us as
// seven launches).
template <int R, bool TRAIN>
__global__ __launch_bounds__(row_threads(R)) void mlp_rows_kernel(const float *raw, const float *labels, MlpBufs m, MlpConst c,
                                                       int bsz, int n_tiles, float inv_n, float *prob)
{
    constexpr bool HALF = R == 8;
    constexpr int NT = row_threads(R), CB = 1024 / NT;                // threads; 16-column blocks of a wave
    constexpr int NI = HALF ? 1 : R / 16, NJ = HALF ? 1 : CB;  // the lane's row and column blocks
    __shared__ __bf16 act[2][R][ACT_LD];
    __shared__ float xs[R][6], ys[R], dl[R];
    __shared__ float pl[10][H];  // W1 by input, b1, b2, b3, W4: read beside weight loads in flight
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    // the lane's values of a layer: columns n0 + 16 j, rows r0 + 16 i + r (r < 4)
    const int n0 = 16 * CB * wave + lr + (HALF ? 16 * (lg >> 1) : 0);
    const int r0 = HALF ? 4 * (lg & 1) : 4 * lg;
    const int64_t ld = m.ld;
    const float *th = m.theta;

    bf16x8 wa[CB][8], wb[CB][8];
    auto load_w = [&](const __bf16 *w, bf16x8 (&f)[CB][8], int t0, int t1) {  // k blocks t0 .. t1 - 1
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int j = 0; j < CB; ++j)
                if (t >= t0 && t < t1) f[j][t] = *(const bf16x8 *)(w + ((CB * wave + j) * 8 + t) * 512 + lane * 8);
    };
    f32x4 acc[NI][NJ];
    auto product = [&](const __bf16 (*in)[ACT_LD], const bf16x8 (&f)[CB][8]) {
        f32x4 s[NI][CB];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) s[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 8; ++t) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const bf16x8 a = *(const bf16x8 *)&in[16 * i + (HALF ? lr & 7 : lr)][32 * t + 8 * lg];
#pragma unroll
                for (int j = 0; j < CB; ++j) s[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, f[j][t], s[i][j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = HALF && lg >= 2 ? s[i][CB - 1][r] : s[i][j][r];
    };
    f32x4 z[3][NI][NJ], e1[3][NI][NJ];
    // nw: a weight matrix to load into f on the way, a few loads a value (a wave that
    // issues them all at once waits for the queue)
    auto activate = [&](int l, __bf16 (*out)[ACT_LD], __bf16 *glob, int b0, const __bf16 *nw, bf16x8 (&f)[CB][8]) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                bf16x4 a;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = r0 + 16 * i + r;
                    if (nw && i == 0 && j == 0) load_w(nw, f, 2 * r, 2 * r + 2);
                    e1[l][i][j][r] = erf1(z[l][i][j][r]);
                    a[r] = (__bf16)gelu(z[l][i][j][r], e1[l][i][j][r]);
                    if (l == 0 && b0 + row >= bsz) a[r] = (__bf16)0.f;
                    out[row][n0 + 16 * j] = a[r];
                }
                if (TRAIN) {
                    const int n = n0 + 16 * j, b = b0 + r0 + 16 * i;
                    *(bf16x4 *)(glob + (l < 2 ? unit_frag(n, b, ld) : unit_col(n, b, ld))) = a;
                }
            }
    };
    auto bias_add = [&](int l) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const float bj = pl[6 + l][n0 + 16 * j];
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) z[l][i][j][r] = acc[i][j][r] + bj;
        }
    };
    // dZ of a layer from d (acc): dZ = d gelu'(Z), to LDS and to memory
    auto derive = [&](int l, __bf16 (*out)[ACT_LD], float *gf, __bf16 *gb, int b0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                f32x4 d;
                bf16x4 db;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = r0 + 16 * i + r;
                    d[r] = acc[i][j][r] * gelu_grad(z[l][i][j][r], e1[l][i][j][r]);
                    if (l == 2 && b0 + row >= bsz) d[r] = 0.f;
                    db[r] = (__bf16)d[r];
                    if (out) out[row][n0 + 16 * j] = db[r];
                }
                const int n = n0 + 16 * j, b = b0 + r0 + 16 * i;
                *(f32x4 *)(gf + unit_col(n, b, ld)) = d;
                if (gb) *(bf16x4 *)(gb + unit_frag(n, b, ld)) = db;
            }
    };
    // Thread 8 row + i < 8 R: input i of a row of the tile at b0 (i = 6: its label)
    float in = 0.f;
    auto input_load = [&](int b0) {
        const int i = tid & 7, b = b0 + (tid >> 3);
        if (tid < 8 * R && b < bsz && i < (TRAIN ? 7 : 6)) {
            const int64_t s = sample_index(b, c);
            in = i < 6 ? raw[s * 6 + i] : labels[s];
        }
    };
    auto input_store = [&](int b0) {
        const int row = tid >> 3, i = tid & 7, b = b0 + row;
        if (tid < 8 * R && i < 6) {
            const float x = b < bsz ? feature(in, i, c) : 0.f;
            xs[row][i] = x;
            if (TRAIN) m.x[i * ld + b] = x;
        } else if (TRAIN && tid < 8 * R && i == 6) {
            ys[row] = in;
        }
    };

    // The tiles of an XCD (workgroups b, b + 8, ...) lie side by side: its L2
    // joins their pieces of lines.
    int tile = blockIdx.x;  // below n_tiles
    if (TRAIN && n_tiles % 8 == 0) tile = (tile % 8) * (n_tiles / 8) + tile / 8;
    // inputs, parameters, weights: loads return in order, so the first two are
    // waited for with the weights in flight
    input_load(tile * R);
    constexpr int NP = (10 * H + NT - 1) / NT;
    float pv[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int q = tid + NT * u, l = q / H;
        if (l < 10)
            pv[u] = th[l < 7 ? q : (l == 7 ? MLP_OFF_W2 + H * H : l == 8 ? MLP_OFF_W3 + H * H : MLP_OFF_W4) + q % H];
    }
    const float b4 = th[MLP_OFF_W4 + H];
    __builtin_amdgcn_sched_barrier(0);
    load_w(m.w2b, wa, 0, 8);
    if (!TRAIN) load_w(m.w3b, wb, 0, 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int q = tid + NT * u, l = q / H;
        if (l < 6) pl[q % 6][q / 6] = pv[u];
        else if (l < 10) pl[l][q % H] = pv[u];
    }
    input_store(tile * R);
    float zo;  // the wave's row's logit
    for (;;) {
        const int b0 = tile * R;
        __syncthreads();
        if (!TRAIN && tile + (int)gridDim.x < n_tiles) input_load((tile + gridDim.x) * R);
        {
            float w1[NJ][7];
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int q = 0; q < 7; ++q) w1[j][q] = pl[q][n0 + 16 * j];
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = r0 + 16 * i + r;
                    float x[6];
#pragma unroll
                    for (int q = 0; q < 6; ++q) x[q] = xs[row][q];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        float v = w1[j][6];
#pragma unroll
                        for (int q = 0; q < 6; ++q) v += w1[j][q] * x[q];
                        z[0][i][j][r] = b0 + row < bsz ? v : 0.f;
                    }
                }
        }
        activate(0, act[0], m.a1, b0, TRAIN ? m.w3b : nullptr, wb);
        __syncthreads();
        product(act[0], wa);
        bias_add(1);
        activate(1, act[1], m.a2, b0, TRAIN ? m.w3t : nullptr, wa);
        __syncthreads();
        product(act[1], wb);
        bias_add(2);
        activate(2, act[0], m.a3, b0, TRAIN ? m.w2t : nullptr, wb);
        __syncthreads();
        if (!TRAIN && tile + (int)gridDim.x < n_tiles) input_store((tile + gridDim.x) * R);
        // output layer and sigmoid, a row a wave (R waves)
        const bool live = b0 + wave < bsz;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < H; i += 64) s += pl[9][i + lane] * (float)act[0][wave][i + lane];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        zo = s + b4;
        const float p = 1.f / (1.f + expf(-zo));
        if (TRAIN) {
            const float d = live ? (p - ys[wave]) * inv_n : 0.f;
            if (lane == 0) {
                dl[wave] = d;
                if (live) m.dlogit[b0 + wave] = d;
            }
            break;
        }
        if (lane == 0 && live) prob[b0 + wave] = p;
        tile += gridDim.x;
        if (tile >= n_tiles) return;
    }
    if (!TRAIN) return;
    const int b0 = tile * R;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const float w4 = pl[9][n0 + 16 * j];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = dl[r0 + 16 * i + r] * w4;
    }
    derive(2, act[1], m.dz3, m.dz3b, b0);
    __syncthreads();
    product(act[1], wa);
    derive(1, act[0], m.dz2, m.dz2b, b0);
    __syncthreads();
    product(act[0], wb);
    derive(0, nullptr, m.dz1, nullptr, b0);
    if (lane == 0 && b0 + wave < bsz) m.lossv[b0 + wave] = fmaxf(zo, 0.f) - zo * ys[wave] + log1pf(expf(-fabsf(zo)));
}

// Adam (Kingma and Ba 2015, bias-corrected); off: the gradient is stored instead.
struct AdamArgs {
    bool on;
    float lr, b1, b2, eps, c1, c2;
};

// A parameter and its moments, loaded ahead of the gradient.
struct AdamState {
    float t, m, v;
};
__device__ __forceinline__ AdamState adam_load(const MlpBufs &m, const AdamArgs &ad, int i)
{
    if (!ad.on) return {};
    return {m.theta[i], m.m[i], m.v[i]};
}

// Finishes parameter i, whose gradient is gi; returns its new value.
__device__ __forceinline__ float adam_step(const MlpBufs &m, const AdamArgs &ad, const AdamState &st, int i, float gi)
{
    if (!ad.on) {
        m.grad[i] = gi;
        return 0.f;
    }
    const float mi = ad.b1 * st.m + (1.f - ad.b1) * gi;
    const float vi = ad.b2 * st.v + (1.f - ad.b2) * gi * gi;
    m.m[i] = mi;
    m.v[i] = vi;
    const float t = st.t - ad.lr * (mi / ad.c1) / (sqrtf(vi / ad.c2) + ad.eps);
    m.theta[i] = t;
    return t;
}

// Every parameter's gradient and update.  Workgroups by blockIdx:
//   [0, 128)    32 x 32 tiles of W2 and W3: wave z forms slice z of the product
//               over the batch, the slices are added in order
//   [128, 320)  8 columns of one section of column sums (three inputs of W1; the
//               other three; b1; b2; b3; W4 and b4), from LDS: a thread sums rows
//               b0 + w, b0 + w + 4, ... of a chunk of MLP_RED_ROWS, the four w are
//               added in order, then the chunks in order
//   320         the batch's mean loss
// All of them run at once; the time is that of the batch's 11 MB coming
// from memory and the last sums (2048 rows: 9.5 us, 26 us as
// four launches).  The tiles
// of an XCD (workgroups b, b + 8, ...) are a 4 x 4 square of one matrix, whose
// operand rows its L2 holds.
constexpr int UPD_W = 128, UPD_C = 192;
// chunks a pass; a chunk in LDS (a wave's 16 chunks x 4 rows on 64 banks); an array
constexpr int UPD_CH = 16, UPD_LD = MLP_RED_ROWS + 4, UPD_QS = UPD_CH * UPD_LD + 4;

__global__ __launch_bounds__(512) void mlp_update_kernel(MlpBufs m, int bsz, int m_pad, int n_slices, int k_slice,
                                                         float inv_n, AdamArgs ad)
{
    __shared__ float sh[11 * UPD_QS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t ld = m.ld;
    if (blockIdx.x < UPD_W) {
        const int xcd = blockIdx.x & 7, t16 = blockIdx.x >> 3;
        const bool w3 = xcd >= 4;
        const int o0 = ((xcd >> 1 & 1) * 4 + (t16 >> 2)) * 32, i0 = ((xcd & 1) * 4 + (t16 & 3)) * 32;
        const __bf16 *A = (w3 ? m.dz3b : m.dz2b) + unit_frag(o0, 0, ld) + lane * 8;
        const __bf16 *B = (w3 ? m.a2 : m.a1) + unit_frag(i0, 0, ld) + lane * 8;
        f32x4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        int par[2];
        AdamState st[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            par[h] = (w3 ? MLP_OFF_W3 : MLP_OFF_W2) + (o0 + (tid >> 5) + 16 * h) * H + i0 + (tid & 31);
            st[h] = adam_load(m, ad, par[h]);
        }
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
                        a[t][i] = *(const bf16x8 *)(A + 16 * i * ld + 16 * (k + 32 * t));
                        b[t][i] = *(const bf16x8 *)(B + 16 * i * ld + 16 * (k + 32 * t));
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
                        sh[(wave * 32 + 16 * i + 4 * (lane >> 4) + r) * 33 + 16 * j + (lane & 15)] = acc[i][j][r];
        }
        __syncthreads();
        __bf16 *wf = w3 ? m.w3b : m.w2b, *wt = w3 ? m.w3t : m.w2t;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int o = (tid >> 5) + 16 * h, i = tid & 31;
            float gi = 0.f;
            for (int z = 0; z < n_slices; ++z) gi += sh[(z * 32 + o) * 33 + i];
            const float t = adam_step(m, ad, st[h], par[h], gi);
            if (!ad.on) continue;
            wf[frag_pos(o0 + o, i0 + i)] = (__bf16)t;
            wt[frag_pos(i0 + i, o0 + o)] = (__bf16)t;
        }
    } else if (blockIdx.x < UPD_W + UPD_C) {
        const int sec = (blockIdx.x - UPD_W) >> 5, j0 = ((blockIdx.x - UPD_W) & 31) * 8;
        const int n_chunks = (bsz + MLP_RED_ROWS - 1) / MLP_RED_ROWS;
        constexpr int V = UPD_CH * MLP_RED_ROWS / 4, NV = (11 * V + 511) / 512;
        // array q of the section: the 8 columns, then x or dlogit
        const int n_arr = sec < 2 ? 11 : sec == 5 ? 9 : 8;
        const float *dz = sec < 3 ? m.dz1 : sec == 3 ? m.dz2 : m.dz3;
        const float *x0 = sec == 5 ? m.dlogit : m.x + 3 * sec * ld;
        // the pass's piece v of four rows: arrays q < 8 are held 8 units by 4 rows
        auto piece = [&](int v, int &q, int &b) {
            q = v < 8 * V ? v & 7 : v / V;
            b = 4 * (v < 8 * V ? v >> 3 : v % V);
        };
        auto fetch = [&](int q, int b) {  // rows b .. b + 3, zero past the batch
            f32x4 v;
            if (sec == 5 && q < 8) {
                const bf16x4 a = *(const bf16x4 *)(m.a3 + unit_col(j0 + q, b, ld));
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (float)a[r];
            } else {
                v = *(const f32x4 *)(q < 8 ? dz + unit_col(j0 + q, b, ld) : x0 + (q - 8) * ld + b);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (b + r >= bsz) v[r] = 0.f;
            return v;
        };
        const int n_ent = sec < 2 ? 3 : sec == 5 ? 2 : 1;
        // the thread's sums: column col, chunk ch of a pass, rows w mod 4
        const int col = tid >> 6, ch = tid >> 2 & 15, w = tid & 3;
        // and its entry in the end: thread 8 e + col finishes entry e of column j
        const int e_end = tid >> 3, j_end = j0 + (tid & 7);
        const bool ends = e_end < n_ent && !(sec == 5 && e_end == 1 && j_end != 0);
        const int par = sec < 2    ? 6 * j_end + 3 * sec + e_end
                        : sec == 2 ? 6 * H + j_end
                        : sec == 3 ? MLP_OFF_W2 + H * H + j_end
                        : sec == 4 ? MLP_OFF_W3 + H * H + j_end
                                   : MLP_OFF_W4 + (e_end == 0 ? j_end : H);
        AdamState st{};
        if (ends) st = adam_load(m, ad, par);
        f32x4 nxt[NV];
        auto fetch_pass = [&](int c0) {
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                int q, b;
                piece(tid + 512 * u, q, b);
                b += c0 * MLP_RED_ROWS;
                nxt[u] = f32x4{0.f, 0.f, 0.f, 0.f};  // zero past the batch
                if (q < n_arr && b < bsz) nxt[u] = fetch(q, b);
            }
        };
        fetch_pass(0);
        float sum = 0.f;
        for (int c0 = 0; c0 < n_chunks; c0 += UPD_CH) {
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                int q, b;
                piece(tid + 512 * u, q, b);
                if (q < n_arr) *(f32x4 *)&sh[q * UPD_QS + b / MLP_RED_ROWS * UPD_LD + b % MLP_RED_ROWS] = nxt[u];
            }
            __syncthreads();
            if (c0 + UPD_CH < n_chunks) fetch_pass(c0 + UPD_CH);
            float t[3] = {0.f, 0.f, 0.f};
            const float *d = sh + col * UPD_QS + ch * UPD_LD + w, *x = sh + 8 * UPD_QS + ch * UPD_LD + w;
            if (sec < 2) {
#pragma unroll
                for (int b = 0; b < MLP_RED_ROWS; b += 4)
#pragma unroll
                    for (int e = 0; e < 3; ++e) t[e] += d[b] * x[e * UPD_QS + b];
            } else if (sec == 5) {
#pragma unroll
                for (int b = 0; b < MLP_RED_ROWS; b += 4) {
                    t[0] += x[b] * d[b];
                    t[1] += x[b];
                }
            } else {
#pragma unroll
                for (int b = 0; b < MLP_RED_ROWS; b += 4) t[0] += d[b];
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                if (e >= n_ent) break;
                const float t1 = __shfl_down(t[e], 1, 4), t2 = __shfl_down(t[e], 2, 4), t3 = __shfl_down(t[e], 3, 4);
                if (w == 0) sh[ch * 24 + 8 * e + col] = ((t[e] + t1) + t2) + t3;
            }
            __syncthreads();
            if (tid < 8 * n_ent) {
                float v[UPD_CH];
#pragma unroll
                for (int q = 0; q < UPD_CH; ++q) v[q] = sh[q * 24 + tid];
#pragma unroll
                for (int q = 0; q < UPD_CH; ++q)
                    if (c0 + q < n_chunks) sum += v[q];
            }
            __syncthreads();
        }
        if (ends) adam_step(m, ad, st, par, sum);
    } else {
        if (tid < 256) {
            float t = 0.f;
#pragma unroll 8
            for (int b = tid; b < bsz; b += 256) t += m.lossv[b];
            sh[tid] = t;
        }
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) sh[tid] += sh[tid + w];
            __syncthreads();
        }
        if (tid == 0) *m.loss += sh[0] * inv_n;
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

// Rows a workgroup: 8 while that is one round of the 256 CUs (a CU holds one
// workgroup).  32 were slower for queries too: the layers' values left the
// registers beside two matrices (200,000 rows: 473 us a call, with 16 466 us).
static int tile_rows(int n) { return n <= 8 * 256 ? 8 : 16; }

hipError_t mlp_predict(const MlpBufs &m, const float *raw, const MlpConst &c, int n, float *prob, hipStream_t s)
{
    const int rows = tile_rows(n), tiles = (int)(((int64_t)n + rows - 1) / rows);
    auto *kern = rows == 8 ? mlp_rows_kernel<8, false> : mlp_rows_kernel<16, false>;
    hipLaunchKernelGGL(kern, dim3(std::min(tiles, 256)), dim3(row_threads(rows)), 0, s, raw, nullptr, m, c, n, tiles, 0.f, prob);
    return hipGetLastError();
}

// Loss and gradient of samples [c.base, c.base + bsz): the gradient into
// m.grad or, with adam, one Adam step t; the batch's mean loss is added to *m.loss.
hipError_t mlp_step(const MlpBufs &m, const float *raw, const float *labels, const MlpConst &c, int bsz,
                    const MlpAdamStep *adam, hipStream_t s)
{
    const int m_pad = (bsz + 63) / 64 * 64;
    const float inv_n = 1.f / (float)bsz;
    const int rows = tile_rows(m_pad), tiles = m_pad / rows;
    hipLaunchKernelGGL((rows == 8 ? mlp_rows_kernel<8, true> : mlp_rows_kernel<16, true>), dim3(tiles), dim3(row_threads(rows)), 0, s, raw,
                       labels, m, c, bsz, tiles, inv_n, nullptr);
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
