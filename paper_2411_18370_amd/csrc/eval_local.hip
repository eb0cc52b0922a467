// Batch runs with a small local bank (a label campaign's: a few f0 bins around
// a source, a few tens of (f1, sky) pairs in a patch of sky): one workgroup per
// run, one lane per (f1, sky) pair, L consecutive f0 values a lane.
//
// The tracks of such a bank stay within LOCAL_W bins of each other, so a
// SUM_BLOCK block's columns [lo, lo + LOCAL_W) of each row are copied to LDS
// and serve every lane; the position of the lane's first f0 is linear in the
// SFT's (s, v - v0), s = dt - tau,
//   x = T a0 (1 + v0.n) + T f1 (1 + v0.n) s + T a0 (v - v0).n,  a0 = f0 + f1 tau,
// (v0, tau: the block's middle SFT), four FP32 FMAs from LDS broadcasts, and on
// a uniform f0 grid of one bin the others' bins follow it while the run guard
// of the grid kernel holds: with u = fract(x + 1/2) and e = dT g - 1, template
// l has bin floor(x + 1/2) + l whenever u and u + (L - 1) e lie in [m, 1 - m).
// The margin m is the host's eta for the grid plus the estimate's bound
//   1.25 (2^-24 (6 T |f1| s + 10 W + 5 (LOCAL_W + 1)) + W |f1 s|/f0 + 2^-48 f0 T)
//   + (L - 1) dT dv,  W = f0 T dv, dv >= |v - v0|
// (terms: roundings of the spindown and velocity terms and of sums up to
// LOCAL_W + 1, the product of both, FP64, and g's change within the block).
// A step where a lane fails takes the canonical FP64 bins (3% of them), a block
// whose columns do not fit the window or the table takes them from the table,
// range-checked.
//
// Per block: windows two blocks ahead stream into a ring of three, the SFTs'
// parameters are formed by the first wave four blocks ahead, every wave adds
// its lanes' bin range three ahead; one barrier a block.
//
// eval_batch_small_kernel, which serves the other small runs, forms every bin
// in FP64 (50 vector instructions a step) and gathers from the table (80 cache
// accesses a step, 65% of its time).  1024 runs x 880 templates x 10^4 SFTs:
// 5.0 ms there, 1.8 ms here (vector units busy 61% of the time, LDS 46%, three
// waves a SIMD of which half wait).
#include "ft_internal.h"

namespace ft {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int LOCAL_THREADS = 256, LOCAL_WAVES = LOCAL_THREADS / 64, RING = 8;

template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_const(const T *p)
{
    return (const __attribute__((address_space(4))) T *)p;
}

struct LocalBlock {
    double v[3], tau;  // of the middle SFT
    float dv, ds;      // bounds of |v - v0| and |s|
};

struct LocalShared {
    float win[3][SUM_BLOCK][LOCAL_W];
    f32x4 par[RING][SUM_BLOCK];
    LocalBlock blk[RING];
    int lo[2][LOCAL_WAVES], hi[2][LOCAL_WAVES];
    int item;
};

// f over the lanes of a wave (f(x, x) = x), by moves between lanes of the vector
// unit: a shuffle goes through LDS, 130 cycles each in a chain of six.
template <int CTRL, int ROWS>
__device__ __forceinline__ int lane_move(int x)
{
    return __builtin_amdgcn_update_dpp(x, x, CTRL, ROWS, 0xf, false);
}
template <typename F>
__device__ __forceinline__ int wave_reduce(int x, F f)
{
    x = f(x, lane_move<0x111, 0xf>(x));  // row_shr 1, 2, 4, 8: rows of 16
    x = f(x, lane_move<0x112, 0xf>(x));
    x = f(x, lane_move<0x114, 0xf>(x));
    x = f(x, lane_move<0x118, 0xf>(x));
    x = f(x, lane_move<0x142, 0xa>(x));  // row_bcast 15 and 31
    x = f(x, lane_move<0x143, 0xc>(x));
    return __builtin_amdgcn_readlane(x, 63);
}
__device__ __forceinline__ int wave_min(int x) { return wave_reduce(x, [](int a, int b) { return min(a, b); }); }
__device__ __forceinline__ int wave_max(int x) { return wave_reduce(x, [](int a, int b) { return max(a, b); }); }
// of floats that are not negative: their bits order like them
__device__ __forceinline__ float wave_maxf(float x) { return __int_as_float(wave_max(__float_as_int(x))); }

__device__ __forceinline__ double read_lane(double x, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// The canonical bins of one step, read from the table.
template <int L>
__device__ __attribute__((noinline)) bool local_canonical(const float *row, const double *f0, const double *v, double dt,
                                                          double f1, double nx, double ny, double nz, double T, int n_i,
                                                          int first_bin, int n_bins, float *val)
{
    const double g = doppler_factor(v[0], v[1], v[2], nx, ny, nz), c = f1 * dt;
    bool bad = false;
    for (int l = 0; l < L; ++l) {
        const int col = bin_fp64(f0[min(l, n_i - 1)], c, g, T) - first_bin;
        bad |= col < 0 || col >= n_bins;
        val[l] = row[min(max(col, 0), n_bins - 1)];
    }
    return bad;
}

template <int L>
__global__ __launch_bounds__(LOCAL_THREADS, 4) void eval_batch_local_kernel(const EvalRun *__restrict__ runs,
                                                                            const int2 *__restrict__ items, int n_items,
                                                                            unsigned *counter)
{
    __shared__ LocalShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (;;) {
        __syncthreads();  // every thread has read the last item and is done with its blocks
        if (tid == 0) sh.item = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(sh.item);
        if (item >= n_items) return;
        const int2 it = items[item];
        EvalRun r = runs[__builtin_amdgcn_readfirstlane(it.x)];
        int chunk = __builtin_amdgcn_readfirstlane(it.y);
        if (r.seg_blocks > 0) {  // split: chunk * rows + row
            const int rows = run_rows(r);
            take_row(r, chunk % rows);
            chunk /= rows;
        }
        const int n_js = r.n_f1 * r.n_sky, n_jsc = (n_js + LOCAL_THREADS - 1) / LOCAL_THREADS;
        const int i0 = chunk / n_jsc * L, n_i = min(L, r.n_f0 - i0);
        const int js_raw = chunk % n_jsc * LOCAL_THREADS + tid;
        const bool live = js_raw < n_js;
        const bool wave_live = __builtin_amdgcn_ballot_w64(live) != 0;  // the others copy windows
        const int js = live ? js_raw : n_js - 1;
        const double f1 = r.f1[js % r.n_f1];
        const double *n = r.sky + 3 * (int64_t)(js / r.n_f1);
        const double nx = n[0], ny = n[1], nz = n[2];
        const double f0 = as_const(r.f0)[i0], span = (as_const(r.f0)[i0 + n_i - 1] - f0) * r.t_sft;
        const double T = r.t_sft;
        const int n_blk = (r.n_sft + SUM_BLOCK - 1) / SUM_BLOCK;

        double raw[4] = {0.0, 0.0, 0.0, 0.0};  // lane k < 32 of the first wave: v and dt of a block's SFT k
        auto load_raw = [&](int b) {
            if (tid < SUM_BLOCK && b < n_blk) {
                const int k = min(b * SUM_BLOCK + tid, r.n_sft - 1);
#pragma unroll
                for (int d = 0; d < 3; ++d) raw[d] = r.v[3 * (int64_t)k + d];
                raw[3] = r.dt[k];
            }
        };
        auto put_par = [&](int b) {
            if (wave != 0 || b >= n_blk) return;
            double mid[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) mid[d] = read_lane(raw[d], SUM_BLOCK / 2);
            f32x4 c;
            c[0] = (float)(raw[3] - mid[3]);
#pragma unroll
            for (int d = 0; d < 3; ++d) c[d + 1] = (float)(raw[d] - mid[d]);
            const bool in = tid < SUM_BLOCK;
            const float dv = wave_maxf(in ? fabsf(c[1]) + fabsf(c[2]) + fabsf(c[3]) : 0.f), ds = wave_maxf(in ? fabsf(c[0]) : 0.f);
            if (tid < SUM_BLOCK) sh.par[b % RING][tid] = c;
            if (tid == 0) {
                LocalBlock &q = sh.blk[b % RING];
#pragma unroll
                for (int d = 0; d < 3; ++d) q.v[d] = mid[d];
                q.tau = mid[3];
                q.dv = dv * (1.f + 0x1p-20f);
                q.ds = ds * (1.f + 0x1p-20f);
            }
        };
        // bins of the wave's lanes in block b, one to spare on either side
        auto window = [&](int b) {
            if (b >= n_blk) return;
            const LocalBlock &q = sh.blk[b % RING];
            const double g = 1.0 + fma(nz, q.v[2], fma(ny, q.v[1], nx * q.v[0]));
            const double aT = fma(f1, q.tau, f0) * T, w = (aT * (double)q.dv + fabs(f1) * (double)q.ds * T) * 1.001;
            const int lo = wave_min((int)floor(fma(aT, g, 0.5 - w)) - 1), hi = wave_max((int)floor(fma(aT + span, g, 0.5 + w)) + 1);
            if (lane == 0) {
                sh.lo[b & 1][wave] = lo;
                sh.hi[b & 1][wave] = hi;
            }
        };
        // first column of block b's window, or -1; issues its copies
        auto stage = [&](int b) -> int {
            if (b >= n_blk) return -1;
            int lo = sh.lo[b & 1][0], hi = sh.hi[b & 1][0];
#pragma unroll
            for (int w = 1; w < LOCAL_WAVES; ++w) {
                lo = min(lo, sh.lo[b & 1][w]);
                hi = max(hi, sh.hi[b & 1][w]);
            }
            lo = __builtin_amdgcn_readfirstlane(lo);
            hi = __builtin_amdgcn_readfirstlane(hi);
            if (lo < r.first_bin || hi >= r.first_bin + r.n_bins || hi - lo >= LOCAL_W) return -1;
            const int col = min(lo - r.first_bin + lane, r.n_bins - 1);
#pragma unroll
            for (int i = 0; i < SUM_BLOCK / LOCAL_WAVES; ++i) {
                const int k = wave + i * LOCAL_WAVES;
                const float *row = r.power_w + (int64_t)min(b * SUM_BLOCK + k, r.n_sft - 1) * r.n_bins;
                __builtin_amdgcn_global_load_lds(row + col, &sh.win[b % 3][k][0], 4, 0, 0);
            }
            return lo;
        };

        float acc[L];
        double tot[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            acc[l] = 0.f;
            tot[l] = 0.0;
        }
        bool bad = false;
        // the ring's start: parameters of blocks 0..3, ranges of 0..2, windows of 0 and 1
#pragma unroll 1
        for (int b = 0; b < 4; ++b) {
            load_raw(b);
            put_par(b);
        }
        load_raw(4);
        __syncthreads();
        window(0);
        window(1);
        __syncthreads();
        int lo = stage(0), lo1 = stage(1);
        __syncthreads();
        window(2);
        for (int b = 0; b < n_blk; ++b) {
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this block's window, issued two blocks ago
            __syncthreads();
            const int lo2 = stage(b + 2);
            put_par(b + 4);
            load_raw(b + 5);
            window(b + 3);
            if (wave_live) {
                const int k0 = b * SUM_BLOCK, len = min(SUM_BLOCK, r.n_sft - k0);
                const LocalBlock &q = sh.blk[b % RING];
                const double g = 1.0 + fma(nz, q.v[2], fma(ny, q.v[1], nx * q.v[0]));
                const double aT = fma(f1, q.tau, f0) * T, dv = (double)q.dv, sT = fabs(f1) * (double)q.ds * T;
                const double W = aT * dv, run = (double)(n_i - 1);
                const double m = r.eta + 1.25 * (0x1p-24 * (6.0 * sT + 10.0 * W + 5.0 * (LOCAL_W + 1)) + dv * sT + 0x1p-48 * aT) +
                                 1e-9 + run * r.dT * dv;
                const double eL = n_i > 1 ? run * (r.dT * g - 1.0) : 0.0;
                const double ulo = m + fmax(0.0, -eL), uhi = (1.0 - m) - fmax(0.0, eL);
                const float w = (float)((uhi - ulo) * (1.0 - 0x1p-22));
                const float c0 = (float)((fma(aT, g, 0.5) - ulo) - (double)lo), c1 = (float)(f1 * T * g);
                const float gx = (float)(aT * nx), gy = (float)(aT * ny), gz = (float)(aT * nz);
                const float *wl = &sh.win[b % 3][0][0];
                auto canonical = [&](int k) {
                    float v[L];
                    bad |= local_canonical<L>(r.power_w + (int64_t)(k0 + k) * r.n_bins, r.f0 + i0, r.v + 3 * (int64_t)(k0 + k),
                                              r.dt[k0 + k], f1, nx, ny, nz, T, n_i, r.first_bin, r.n_bins, v);
#pragma unroll
                    for (int l = 0; l < L; ++l) acc[l] += v[l];
                };
                if (lo < 0) {
#pragma unroll 1
                    for (int k = 0; k < len; ++k) canonical(k);
                } else {
#pragma unroll 1
                    for (int k = 0; k < len; k += 4) {
                        float v[4][L];
                        float fr[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {  // rows past the last SFT repeat it
                            const f32x4 c = sh.par[b % RING][k + i];
                            float x = __builtin_fmaf(c[0], c1, c0);
                            x = __builtin_fmaf(c[1], gx, x);
                            x = __builtin_fmaf(c[2], gy, x);
                            x = __builtin_fmaf(c[3], gz, x);
                            fr[i] = __builtin_amdgcn_fractf(x);
                            const float *at = wl + (k + i) * LOCAL_W + (int)x;
#pragma unroll
                            for (int l = 0; l < L; ++l) v[i][l] = at[l];
                        }
                        if (__builtin_amdgcn_ballot_w64(!(fmaxf(fmaxf(fr[0], fr[1]), fmaxf(fr[2], fr[3])) < w)) != 0) {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (__builtin_amdgcn_ballot_w64(!(fr[i] < w)) != 0) {
                                    const int q = min(k0 + k + i, r.n_sft - 1);
                                    const auto *vk = as_const(r.v + 3 * (int64_t)q);
                                    const double gk = doppler_factor(vk[0], vk[1], vk[2], nx, ny, nz), ck = f1 * as_const(r.dt)[q];
#pragma unroll
                                    for (int l = 0; l < L; ++l)
                                        v[i][l] = wl[(k + i) * LOCAL_W + bin_fp64(as_const(r.f0)[i0 + min(l, n_i - 1)], ck, gk, T) - lo];
                                }
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if (k + i >= len) break;
#pragma unroll
                            for (int l = 0; l < L; ++l) acc[l] += v[i][l];
                        }
                    }
                }
                if (r.bsum) {
                    float *out = r.bsum + (int64_t)b * r.bsum_n + (int64_t)js * r.n_f0 + i0;
#pragma unroll
                    for (int l = 0; l < L; ++l) {
                        if (live && l < n_i) out[l] = acc[l];
                        acc[l] = 0.f;
                    }
                } else if (r.sum_mode == FT_SUM_BLOCKED) {
#pragma unroll
                    for (int l = 0; l < L; ++l) {
                        tot[l] += (double)acc[l];
                        acc[l] = 0.f;
                    }
                }
            }
            lo = lo1;
            lo1 = lo2;
        }
        if (bad && live) atomicOr(r.err, ERR_RANGE);
        if (live && !r.bsum) {
            float *out = r.stats + (int64_t)js * r.n_f0 + i0;
#pragma unroll
            for (int l = 0; l < L; ++l)
                if (l < n_i) out[l] = (float)(tot[l] + (double)acc[l]);
        }
    }
}

}  // namespace

hipError_t launch_eval_batch_local(const EvalRun *runs, const int2 *items, int n_items, int f0_chunk, unsigned *counter,
                                   int grid, hipStream_t s)
{
    if (n_items <= 0) return hipSuccess;
    if (f0_chunk != 5 && f0_chunk != 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL((f0_chunk == 5 ? eval_batch_local_kernel<5> : eval_batch_local_kernel<8>), dim3((unsigned)grid),
                       dim3(LOCAL_THREADS), 0, s, runs, items, n_items, counter);
    return hipGetLastError();
}

}  // namespace ft
