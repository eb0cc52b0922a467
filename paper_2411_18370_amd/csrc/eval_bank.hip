// Binary-system banks through LDS windows: one lane per template, the table
// rows of a SUM_BLOCK-SFT block staged in LDS, and the track of each block a
// polynomial in time.  It serves banks whose whole bin range fits an LDS row
// (a search band of a few hundred bins); eval_binary_kernel serves the rest.
//
// Split of the work.  A workgroup takes 512 templates and walks the blocks; the
// windows [win_lo, win_lo + W) of the next block stream into LDS
// (global_load_lds, 16 bytes a lane) while the current one is summed, so a row
// is fetched once per workgroup instead of once per wave-level gather, and the
// gathers are LDS reads at a lane address plus an immediate row offset (W is a
// compile-time row stride).
//
// Track.  A block is cut into segments (a bit mask per block, bit j set where
// SFT j starts one) whose times ascend and span at most 2 hs; nearly every
// block is one segment, those across a data gap or a change of detector are
// more.  With tau the segment's mid-time and s = (dt - tau)/hs in [-1, 1], the
// position in bins is
//   x = f0 T (1 + v(s).n) - C cos(th0 + om1 s),
//   C = f0 T a_p Omega, om1 = Omega hs, th0 = Omega tau - phi_b.
// v(s) is a polynomial of degree 5 fitted to the block's velocities
// (bank_fit_kernel, least squares, residual measured), the cosine its Taylor
// polynomial of the same degree, so x = sum k_j s^j: five FP32 FMAs per SFT,
// with k_0 formed in FP64 less its nearest integer (the whole Doppler shift is
// in k_0; the other terms are a few bins).
//
// Guard.  n = rint(x) in FP32 is the canonical bin whenever |x - n| <
// 1/2 - eps, eps the bound below.  Per SFT only the largest |x - n| is kept; a
// wave whose maximum fails for some lane sums the block again with the check
// per SFT and the canonical FP64 bin (library cosine) where it fails.
// Segments shorter than a block, and blocks whose velocities the polynomial
// does not fit, are summed SFT by SFT with the velocities themselves.
//
// Bound.  With u = 2^-24, X >= |k_1| and Y >= |k_2| + .. + |k_5|: the rounding
// of k_0 u/2, of k_1 and s u X each (dx/ds is k_1 up to 5 Y), of the other
// coefficients 6 u Y and s^j 5 u Y, the Horner steps below 1.2 u Y and the one
// to k_1 u (X + Y), the last FMA u (X + Y + 1/2), x + 1.5 2^23 exact to the
// integer: u (4 X + 15 Y + 1); the per-SFT form with v - v0 adds 6 u W, W = f0 T
// max|v - v0|.  X is C om1 plus the fit's share, Y C om1^2 (0.5 + om1) plus the
// fit's share; the fit's coefficients sum to at most 3 max|v - v0|, a third of
// them beyond the linear one (both are checked).  The Taylor remainder is below
// C om1^6/720 (1 + om1), the FP64 sine and cosine (Taylor to th^9 and th^10 on
// |th| <= pi/4) are within 2e-9, the phase within 2^-50 of its size, k_0 and
// the canonical value within 2^-49 f0 T.  bank_eps adds them and the fit's
// residual (per block) with a margin of 1.25.
//
// What binds it: vector issue, then the barrier a block.  Measured per wave on
// MI355X, an FP32 FMA or add takes 2.8 cycles when every operand is a VGPR and
// 4.8 with an SGPR operand, FP64 and conversions 4.7, a lane-half swap 8.5;
// FP32 MFMAs take their cycles from the same units (the polynomials as 16x16x4
// products: 9.4 ms).  So the s values come from LDS (a broadcast read of four),
// and the bin is found by adding 1.5 2^23 (fast adds) instead of fract and a
// conversion: 14 vector instructions per SFT and template wave against 15.4
// slower ones in the gather kernel.  2e6 templates x 10^4 SFTs (190 bins):
// 13.3 -> 7.4 ms (1.5 -> 2.7e12 evaluations/s); of it 0.35 ms sum blocks again,
// 0.55 ms copy windows, 0.9 ms is the waves' skew at the barriers.  512
// threads with four waves per SIMD: 1024 threads took 9.4 ms (the barrier
// couples more waves), 256 threads 8.5 ms (more copies), five or six waves per
// SIMD with a narrower row 8.0 against 8.07 ms (earlier form).
#include "ft_internal.h"

namespace ft {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_const(const T *p)
{
    return (const __attribute__((address_space(4))) T *)p;
}

// Velocity polynomial of a block: v(s) = v0 + v1 s + sum_{j=2..5} v[j-2] s^j.
struct BankFit {
    double v0[3], v1[3];
    float v[4][3];
    int32_t pad;
    float res;  // residual with the margin of the bound (-1: no fit)
};

// One template, as the canonical bin needs it (aw = a_p Omega), and its
// per-block factors.
struct BankLane {
    double f0, nx, ny, nz, aw, om, phib;
    float q2, q3, q4, q5, thr, f0T;  // thr: 1/2 - eps without a fit's residual
};

constexpr float ROUND_MAGIC = 12582912.f;       // 1.5 2^23: x + magic rounds x to an integer
constexpr uint32_t ROUND_BITS4 = 0x2D000000u;   // 4 times its bit pattern, modulo 2^32

// Taylor coefficients of the segment's sine and cosine, read per segment (as
// literals they would be held in registers across the gathers).
__constant__ double kTrig[8] = {1.0 / 362880,   -1.0 / 5040, 1.0 / 120,  -1.0 / 6,
                                -1.0 / 3628800, 1.0 / 40320, -1.0 / 720, 1.0 / 24};

// Cosine and sine of the orbital phase at offset tau.
__device__ __forceinline__ void bank_phase(const BankLane &p, double tau, double &c, double &s)
{
    const double y = fma(p.om, tau, -p.phib) * 0x1.45f306dc9c883p-3;  // revolutions
    const double yr = y - __builtin_rint(y);
    const double qd = __builtin_rint(4.0 * yr);
    const double th = fma(qd, -0.25, yr) * 0x1.921fb54442d18p+2;
    const double z = th * th;
    const auto *kt = as_const(kTrig);
    asm volatile("" : "+s"(kt));
    double ps = fma(z, kt[0], kt[1]);
    ps = fma(z, ps, kt[2]);
    ps = fma(z, ps, kt[3]);
    const double sn = fma(th * z, ps, th);
    double pc = fma(z, kt[4], kt[5]);
    pc = fma(z, pc, kt[6]);
    pc = fma(z, pc, kt[7]);
    pc = fma(z, pc, -0.5);
    const double cs = fma(z, pc, 1.0);
    const int n = (int)qd & 3;
    // quadrant n: (cos, sin) = (cs, sn), (-sn, cs), (-cs, -sn), (sn, -cs)
    const double cu = n & 1 ? sn : cs, su = n & 1 ? cs : sn;
    c = __hiloint2double(__double2hiint(cu) ^ (((n + 1) & 2) << 30), __double2loint(cu));
    s = __hiloint2double(__double2hiint(su) ^ ((n & 2) << 30), __double2loint(su));
}

// k_0 .. k_5 of a segment with mid-time tau and velocity v0 + sum vj s^j (vj
// null: v0 alone); base: LDS byte offset in a row of the column of the integer
// taken out of k_0.  k_1 dominates the others and is summed in FP64.
__device__ __forceinline__ void bank_poly(const BankLane &p, double T, double tau,
                                          const __attribute__((address_space(4))) double *v0,
                                          const __attribute__((address_space(4))) double *v1,
                                          const __attribute__((address_space(4))) float *vj, double hs, int win_lo,
                                          float (&k)[6], int &base)
{
    double c, s;
    bank_phase(p, tau, c, s);
    const double f0T = p.f0 * T;
    const double d = fma(p.nz, v0[2], fma(p.ny, v0[1], p.nx * v0[0]));
    const double A = fma(f0T, fma(-p.aw, c, d), f0T);
    const double ai = __builtin_rint(A);
    const float sf = (float)s, cf = (float)c;
    double e = (p.aw * (p.om * hs)) * s;
    k[0] = (float)(A - ai);
    k[2] = p.q2 * cf;
    k[3] = p.q3 * sf;
    k[4] = p.q4 * cf;
    k[5] = p.q5 * sf;
    if (vj) {
        e = fma(p.nz, v1[2], fma(p.ny, v1[1], fma(p.nx, v1[0], e)));
        const float gx = (float)(f0T * p.nx), gy = (float)(f0T * p.ny), gz = (float)(f0T * p.nz);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            k[j + 2] = __builtin_fmaf(gz, vj[3 * j + 2], __builtin_fmaf(gy, vj[3 * j + 1],
                                                                      __builtin_fmaf(gx, vj[3 * j], k[j + 2])));
    }
    k[1] = (float)(f0T * e);
    base = ((int)ai - win_lo) * 4;
}

__device__ __forceinline__ float horner5(const float (&k)[6], float s)
{
    float t = __builtin_fmaf(s, k[5], k[4]);
    t = __builtin_fmaf(s, t, k[3]);
    t = __builtin_fmaf(s, t, k[2]);
    t = __builtin_fmaf(s, t, k[1]);
    return __builtin_fmaf(s, t, k[0]);
}

// LDS byte addresses: the gathers add a lane's bin to one base per segment and
// take the row from the instruction's immediate offset.
typedef const __attribute__((address_space(3))) float lds_float;
typedef const __attribute__((address_space(3))) f32x4 lds_f32x4;

__device__ __forceinline__ int lds_addr(const float *p) { return (int)(uint32_t)(uintptr_t)(lds_float *)p; }

__device__ __forceinline__ float lds_at(int addr) { return *(lds_float *)(uintptr_t)(uint32_t)addr; }

// Canonical bin of a template at SFT k (the guard's rare fallback; out of line,
// so the library cosine's constants are not held while the blocks are summed).
__device__ __attribute__((noinline)) int bank_canonical(const double *v, const double *dt, double T, double f0, double nx,
                                                        double ny, double nz, double aw, double om, double phib, int k)
{
    const auto *vk = as_const(v + 3 * (int64_t)k);
    return bin_binary(f0, doppler_factor(vk[0], vk[1], vk[2], nx, ny, nz), aw, om, phib, as_const(dt)[k], T);
}

// LDS byte address in the row at `row` of the bin of position x at SFT k, checked.
__device__ __forceinline__ int bank_checked(const EvalRun &r, const BankLane &p, float x, float thr, int base, int row,
                                            int k, int win_lo)
{
    const float n = __builtin_rintf(x);
    int off = (int)n * 4 + base;
    const bool bad = !(__builtin_fabsf(x - n) < thr);
    if (__builtin_amdgcn_ballot_w64(bad) != 0) {
        const int B = bank_canonical(r.v, r.dt, r.t_sft, p.f0, p.nx, p.ny, p.nz, p.aw, p.om, p.phib, k);
        off = bad ? (B - win_lo) * 4 : off;
    }
    return row + off;
}

// Bytes of a window buffer: SUM_BLOCK rows of W columns and the block's s.
template <int W>
constexpr int kBufFloats = SUM_BLOCK * W + SUM_BLOCK;

constexpr int kWaves = BANK_THREADS / 64;

// Table windows of block b into buf: columns [win_lo, win_lo + cols) of each
// row, 16 bytes a lane (cols is a multiple of 4; reads past a row's end take
// the next row's first columns, past the table's end its padding, and no
// template's bin is there; rows past the last SFT repeat it), then the block's
// s.  Wave w takes every kWaves-th row (pairs of rows where two fit a copy)
// from a scalar row base and one lane offset.
template <int W>
__device__ __forceinline__ void bank_stage(const EvalRun &r, const BankPlan &pl, int b, float *buf)
{
    const uint32_t lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int last = min(SUM_BLOCK, r.n_sft - b * SUM_BLOCK) - 1;
    const char *src = (const char *)(r.power_w + (int64_t)b * SUM_BLOCK * r.n_bins + (pl.win_lo - r.first_bin));
    const int64_t pitch = (int64_t)r.n_bins * 4;
    if (W == 128) {
        if ((int)(lane & 31) * 4 < pl.cols) {
#pragma unroll
            for (int i = 0; i < SUM_BLOCK / 2 / kWaves; ++i) {
                const int k = 2 * (wave + i * kWaves);
                const bool two = k < last;
                __builtin_amdgcn_global_load_lds(src + min(k, last) * pitch + (two ? (lane >> 5) * (uint32_t)pitch : 0u) +
                                                     (lane & 31) * 16u, buf + k * W, 16, 0, 0);
            }
        }
    } else {
#pragma unroll
        for (int x = 0; x < W; x += 256)
            if (x + (int)lane * 4 < pl.cols) {
#pragma unroll
                for (int i = 0; i < SUM_BLOCK / kWaves; ++i) {
                    const int k = wave + i * kWaves;
                    __builtin_amdgcn_global_load_lds(src + (min(k, last) * pitch + x * 4) + lane * 16u, buf + k * W + x, 16, 0, 0);
                }
            }
    }
    if (wave == 0 && lane < SUM_BLOCK / 4)
        __builtin_amdgcn_global_load_lds((const char *)(pl.sval + b * SUM_BLOCK) + lane * 16u, buf + SUM_BLOCK * W, 16, 0, 0);
}

// SPLIT: workgroup row y takes blocks [y bps, (y + 1) bps) and stores every
// block's FP32 sum in bsum[block][template] (added in block order by
// block_sum_kernel: the unsplit kernel's sequence of operations).
template <int W, bool SPLIT>
__global__ __launch_bounds__(BANK_THREADS, 4) void eval_bank_kernel(EvalRun r, BankPlan pl, float *bsum, int bps)
{
    extern __shared__ float win[];  // [2][kBufFloats]
    const int n_blk = (r.n_sft + SUM_BLOCK - 1) / SUM_BLOCK;
    const int b0 = SPLIT ? (int)blockIdx.y * bps : 0;
    const int b1 = SPLIT ? min(b0 + bps, n_blk) : n_blk;
    if (b0 >= b1) return;
    const int64_t t_raw = (int64_t)blockIdx.x * BANK_THREADS + threadIdx.x;
    const bool live = t_raw < r.n_list;
    // waves past the bank's end only copy windows
    const bool wave_live = __builtin_amdgcn_ballot_w64(live) != 0;
    const int64_t t = live ? t_raw : r.n_list - 1;
    bank_stage<W>(r, pl, b0, win);
    BankLane p;
    p.f0 = r.f0[t];
    p.nx = r.sky[3 * t];
    p.ny = r.sky[3 * t + 1];
    p.nz = r.sky[3 * t + 2];
    p.om = r.omega[t];
    p.aw = r.ap[t] * p.om;
    p.phib = r.phib[t];
    {
        const double f0T = p.f0 * r.t_sft, C = f0T * p.aw, o1 = p.om * pl.hs, o2 = o1 * o1;
        const double eps = bank_eps(f0T, C, o1, p.om * pl.dt_abs + fabs(p.phib), pl.dv_max, 0.0);
        // -C cos(th0 + o1 s) + C cos(th0) = sin(th0) C (d - d^3/6 + d^5/120) +
        // cos(th0) C (d^2/2 - d^4/24), d = o1 s
        p.q2 = (float)(C * o2 * 0.5);
        p.q3 = (float)(-(C * o1 * o2 * (1.0 / 6)));
        p.q4 = (float)(-(C * o2 * o2 * (1.0 / 24)));
        p.q5 = (float)(C * o2 * o2 * o1 * (1.0 / 120));
        p.thr = (float)(0.5 - eps) - 0x1p-24f;
        p.f0T = (float)(f0T * (1.0 + 0x1p-22));
    }
    const auto *fit = as_const((const BankFit *)pl.fit);
    float acc = 0.f;
    double tot = 0.0;
    for (int b = b0; b < b1; ++b) {
        // the copies of block b have landed (every wave waits for its own),
        // and every wave is done with the other buffer
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        const int cur = (b - b0) & 1;
        if (b + 1 < b1) bank_stage<W>(r, pl, b + 1, win + (cur ^ 1) * kBufFloats<W>);
        const int wb = lds_addr(win) + cur * kBufFloats<W> * 4;
        const int k0 = b * SUM_BLOCK, len = min(SUM_BLOCK, r.n_sft - k0);
        if (!wave_live) continue;
        if (fit[b].res >= 0.f) {
            float k[6];
            int base;
            bank_poly(p, r.t_sft, 0.5 * (as_const(r.dt)[k0] + as_const(r.dt)[k0 + SUM_BLOCK - 1]), fit[b].v0, fit[b].v1,
                      fit[b].v[0], pl.hs, pl.win_lo, k, base);
            const float thr = __builtin_fmaf(-p.f0T, fit[b].res, p.thr) - 0x1p-24f;
            float a = acc, top = 0.f;
            uint32_t at = (uint32_t)(wb + base) - ROUND_BITS4;
            float magic = ROUND_MAGIC;
            asm("" : "+v"(at), "+v"(magic));  // one base; the constant stays in a VGPR
#pragma unroll
            for (int h = 0; h < SUM_BLOCK; h += 8) {
                float v[8];
                const f32x4 sa = *(lds_f32x4 *)(uintptr_t)(uint32_t)(wb + (SUM_BLOCK * W + h) * 4);
                const f32x4 sb = *(lds_f32x4 *)(uintptr_t)(uint32_t)(wb + (SUM_BLOCK * W + h + 4) * 4);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float x = horner5(k, i < 4 ? sa[i] : sb[i - 4]);
                    const float m = x + magic;
                    top = __builtin_fmaxf(top, __builtin_fabsf(x - (m - magic)));
                    v[i] = lds_at((int)((__float_as_uint(m) << 2) + at) + (h + i) * (W * 4));
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) a += v[i];
            }
            if (__builtin_amdgcn_ballot_w64(!(top < thr)) != 0) {
                a = acc;
#pragma unroll 1
                for (int h = 0; h < SUM_BLOCK; h += 8) {
                    int ad[8];
                    const f32x4 sa = *(lds_f32x4 *)(uintptr_t)(uint32_t)(wb + (SUM_BLOCK * W + h) * 4);
                    const f32x4 sb = *(lds_f32x4 *)(uintptr_t)(uint32_t)(wb + (SUM_BLOCK * W + h + 4) * 4);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        ad[i] = bank_checked(r, p, horner5(k, i < 4 ? sa[i] : sb[i - 4]), thr, base,
                                             wb + (h + i) * W * 4, k0 + h + i, pl.win_lo);
#pragma unroll
                    for (int i = 0; i < 8; ++i) a += lds_at(ad[i]);
                }
            }
            acc = a;
        } else {
            uint32_t m = as_const(pl.mask)[b];
            const f32x4 *par = (const f32x4 *)pl.par;
            while (m) {
                const int f = __builtin_ctz(m);
                m &= m - 1;
                const int kf = k0 + f, kl = k0 + (m ? __builtin_ctz(m) - 1 : len - 1);
                float k[6];
                int base;
                bank_poly(p, r.t_sft, 0.5 * (as_const(r.dt)[kf] + as_const(r.dt)[kl]),
                          as_const(r.v + 3 * (int64_t)((kf + kl) >> 1)), nullptr, nullptr, pl.hs, pl.win_lo, k, base);
                const double f0T = p.f0 * r.t_sft;
                const float gx = (float)(f0T * p.nx), gy = (float)(f0T * p.ny), gz = (float)(f0T * p.nz);
#pragma unroll 1
                for (int q = kf; q <= kl; ++q) {
                    const f32x4 c = as_const(par)[q];
                    float x = horner5(k, c[0]);
                    x = __builtin_fmaf(c[1], gx, x);
                    x = __builtin_fmaf(c[2], gy, x);
                    x = __builtin_fmaf(c[3], gz, x);
                    acc += lds_at(bank_checked(r, p, x, p.thr, base, wb + (q - k0) * W * 4, q, pl.win_lo));
                }
            }
        }
        if (SPLIT) {
            if (live) bsum[(int64_t)b * r.n_list + t] = acc;
            acc = 0.f;
        } else if (r.sum_mode == FT_SUM_BLOCKED) {
            tot += (double)acc;
            acc = 0.f;
        }
    }
    if (!SPLIT && live) r.stats[t] = (float)(tot + (double)acc);
}

// List banks (arbitrary f0, f1, sky) the same way: with a0 = f0 + f1 tau, a1 =
// f1 hs and the segment's v0 the position at an SFT is
//   x = T a0 (1 + v0.n) + T a1 (1 + v0.n) s + T a0 (v - v0).n,
// four FMAs from the SFT's (s, v - v0), which stream into LDS beside the window
// (a1/a0 of the last term is in the bound, list_eps: k_0 and the sums 3 u, their
// terms' roundings 6 u T a1 and 10 u W).  No fit is needed, so blocks may span
// most of a day (32 SFTs of 1800 s; a polynomial there would take degree 9).
//
// Templates are taken in the order of their f0 (list_order_kernel), so a
// workgroup's window is little more than the Doppler range: LIST_W columns hold
// it unless few templates lie far apart; such a workgroup reads the table
// itself, at canonical bins.  Before, one lane a template walked all SFTs with
// a gather and ten FP64 operations in a chain: 2e5 templates (0.25 Hz) x 5000
// SFTs 2.85 ms, now 0.42 ms (2.4e12 evaluations/s; vector units busy 68% of the
// time, LDS 54%, three waves a SIMD of which half wait).
constexpr int LIST_W = 256;
constexpr int kListFloats = kBufFloats<LIST_W> + 4 * SUM_BLOCK;  // the window, s, (s, v - v0)

struct ListLane {
    double f0, f1, nx, ny, nz;
    float thr;
};

// A template in a segment: k_0 less its nearest integer (whose LDS offset is
// base), k_1, and T a0 n.
struct ListSeg {
    float k0, k1, gx, gy, gz;
    int base;
};

// Canonical bin of a list template at SFT k (the guard's rare fallback).
__device__ __forceinline__ int list_canonical(const EvalRun &r, const ListLane &p, int k)
{
    const auto *vk = as_const(r.v + 3 * (int64_t)k);
    return bin_fp64(p.f0, p.f1 * as_const(r.dt)[k], doppler_factor(vk[0], vk[1], vk[2], p.nx, p.ny, p.nz), r.t_sft);
}

// Segment of SFTs [kf, kl].
__device__ __forceinline__ ListSeg list_seg(const EvalRun &r, const ListLane &p, int kf, int kl, double hs, int win_lo)
{
    const double tau = 0.5 * (as_const(r.dt)[kf] + as_const(r.dt)[kl]);
    const auto *v0 = as_const(r.v + 3 * (int64_t)((kf + kl) >> 1));
    const double aT = fma(p.f1, tau, p.f0) * r.t_sft, bT = (p.f1 * hs) * r.t_sft;
    const double d = fma(p.nz, v0[2], fma(p.ny, v0[1], p.nx * v0[0]));
    const double A = fma(aT, d, aT), ai = __builtin_rint(A);
    return {(float)(A - ai),   (float)fma(bT, d, bT), (float)(aT * p.nx),
            (float)(aT * p.ny), (float)(aT * p.nz),    ((int)ai - win_lo) * 4};
}

__device__ __forceinline__ float list_pos(const ListSeg &g, const f32x4 c)
{
    float x = __builtin_fmaf(c[0], g.k1, g.k0);
    x = __builtin_fmaf(c[1], g.gx, x);
    x = __builtin_fmaf(c[2], g.gy, x);
    return __builtin_fmaf(c[3], g.gz, x);
}

// LDS byte address in the row at `row` of the bin of position x at SFT k, checked.
__device__ __forceinline__ int list_checked(const EvalRun &r, const ListLane &p, float x, int base, int row, int k, int win_lo)
{
    const float n = __builtin_rintf(x);
    int off = (int)n * 4 + base;
    const bool bad = !(__builtin_fabsf(x - n) < p.thr);
    if (__builtin_amdgcn_ballot_w64(bad) != 0) {
        const int B = list_canonical(r, p, k);
        off = bad ? (B - win_lo) * 4 : off;
    }
    return row + off;
}

// One SUM_BLOCK block of a lane from its window at LDS address wb; returns the
// running sum.
__device__ __forceinline__ float list_block(const EvalRun &r, const BankPlan &pl, const ListLane &p, int b, int wb, float acc)
{
    constexpr int W = LIST_W;
    const int k0 = b * SUM_BLOCK, len = min(SUM_BLOCK, r.n_sft - k0);
    const int par = wb + (kBufFloats<W>) * 4;
    uint32_t m = as_const(pl.mask)[b];
    if (m == 1u && len == SUM_BLOCK) {
        const ListSeg g = list_seg(r, p, k0, k0 + SUM_BLOCK - 1, pl.hs, pl.win_lo);
        float a = acc, top = 0.f;
        uint32_t at = (uint32_t)(wb + g.base) - ROUND_BITS4;
        float magic = ROUND_MAGIC;
        asm("" : "+v"(at), "+v"(magic));  // one base; the constant stays in a VGPR
#pragma unroll
        for (int h = 0; h < SUM_BLOCK; h += 8) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float x = list_pos(g, *(lds_f32x4 *)(uintptr_t)(uint32_t)(par + (h + i) * 16));
                const float n = x + magic;
                top = __builtin_fmaxf(top, __builtin_fabsf(x - (n - magic)));
                v[i] = lds_at((int)((__float_as_uint(n) << 2) + at) + (h + i) * (W * 4));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) a += v[i];
        }
        if (__builtin_amdgcn_ballot_w64(!(top < p.thr)) == 0) return a;
    }
    // segments shorter than a block, and blocks with a bin to check, SFT by SFT
    while (m) {
        const int f = __builtin_ctz(m);
        m &= m - 1;
        const int kf = k0 + f, kl = k0 + (m ? __builtin_ctz(m) - 1 : len - 1);
        const ListSeg g = list_seg(r, p, kf, kl, pl.hs, pl.win_lo);
#pragma unroll 1
        for (int q = kf; q <= kl; ++q) {
            const f32x4 c = *(lds_f32x4 *)(uintptr_t)(uint32_t)(par + (q - k0) * 16);
            acc += lds_at(list_checked(r, p, list_pos(g, c), g.base, wb + (q - k0) * W * 4, q, pl.win_lo));
        }
    }
    return acc;
}

// Window of block b and its SFTs' (s, v - v0).
__device__ __forceinline__ void list_stage(const EvalRun &r, const BankPlan &pl, int b, float *buf)
{
    bank_stage<LIST_W>(r, pl, b, buf);
    const uint32_t tid = threadIdx.x;
    if (tid >= 64 && tid < 64 + SUM_BLOCK)  // the table is padded to whole blocks
        __builtin_amdgcn_global_load_lds((const char *)(pl.par + (int64_t)b * SUM_BLOCK * 4) + (tid - 64) * 16u,
                                         buf + kBufFloats<LIST_W>, 16, 0, 0);
}

// The same block at canonical bins from the table (windows that do not fit).
__device__ __forceinline__ float list_block_direct(const EvalRun &r, const ListLane &p, int b, float acc)
{
    const int k0 = b * SUM_BLOCK, k1 = min(k0 + SUM_BLOCK, r.n_sft);
    for (int k = k0; k < k1; k += 8) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int q = min(k + i, k1 - 1);
            const int col = min(max(list_canonical(r, p, q) - r.first_bin, 0), r.n_bins - 1);
            v[i] = r.power_w[(int64_t)q * r.n_bins + col];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (k + i < k1) acc += v[i];
    }
    return acc;
}

template <bool SPLIT>
__global__ __launch_bounds__(BANK_THREADS, 4) void eval_list_kernel(EvalRun r, BankPlan pl, const int32_t *order, double dt_lo,
                                                                    double dt_hi, float *bsum, int bps)
{
    extern __shared__ float win[];  // [2][kListFloats]
    __shared__ int lo_w[kWaves], hi_w[kWaves];
    const int n_blk = (r.n_sft + SUM_BLOCK - 1) / SUM_BLOCK;
    const int b0 = SPLIT ? (int)blockIdx.y * bps : 0;
    const int b1 = SPLIT ? min(b0 + bps, n_blk) : n_blk;
    if (b0 >= b1) return;
    const int64_t i_raw = (int64_t)blockIdx.x * BANK_THREADS + threadIdx.x;
    const bool live = i_raw < r.n_list;
    const bool wave_live = __builtin_amdgcn_ballot_w64(live) != 0;  // the others only copy windows
    const int64_t pos = live ? i_raw : r.n_list - 1, t = order[pos];
    ListLane p;
    p.f0 = r.f0[t];
    p.f1 = r.f1[t];
    p.nx = r.sky[3 * t];
    p.ny = r.sky[3 * t + 1];
    p.nz = r.sky[3 * t + 2];
    {
        // bins of the track at any time, two to spare
        const double c0 = p.f1 * dt_lo, c1 = p.f1 * dt_hi, fl = (p.f0 + fmin(c0, c1)) * (1.0 - r.vmax) * r.t_sft,
                     fh = (p.f0 + fmax(c0, c1)) * (1.0 + r.vmax) * r.t_sft;
        int lo = (int)floor(fl + 0.5) - 2, hi = (int)floor(fh + 0.5) + 2;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, __shfl_xor(lo, o, 64));
            hi = max(hi, __shfl_xor(hi, o, 64));
        }
        if ((threadIdx.x & 63) == 0) {
            lo_w[threadIdx.x >> 6] = lo;
            hi_w[threadIdx.x >> 6] = hi;
        }
        const double f0T = (p.f0 + fabs(p.f1) * pl.dt_abs) * r.t_sft, bT = fabs(p.f1) * pl.hs * r.t_sft;
        p.thr = (float)(0.5 - list_eps(f0T, bT, pl.dv_max)) - 0x1p-24f;
    }
    __syncthreads();
    int lo = lo_w[0], hi = hi_w[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
        lo = min(lo, lo_w[w]);
        hi = max(hi, hi_w[w]);
    }
    pl.win_lo = __builtin_amdgcn_readfirstlane(max(lo, r.first_bin));
    const int win_hi = __builtin_amdgcn_readfirstlane(min(hi, r.first_bin + r.n_bins - 1));
    pl.cols = (win_hi - pl.win_lo + 4) & ~3;
    const bool fits = pl.cols <= LIST_W;
    if (fits) list_stage(r, pl, b0, win);
    float acc = 0.f;
    double tot = 0.0;
    for (int b = b0; b < b1; ++b) {
        if (fits) {
            // the copies of block b have landed (every wave waits for its own),
            // and every wave is done with the other buffer
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            __syncthreads();
            const int cur = (b - b0) & 1;
            if (b + 1 < b1) list_stage(r, pl, b + 1, win + (cur ^ 1) * kListFloats);
            if (!wave_live) continue;
            acc = list_block(r, pl, p, b, lds_addr(win) + cur * kListFloats * 4, acc);
        } else {
            if (!wave_live) continue;
            acc = list_block_direct(r, p, b, acc);
        }
        if (SPLIT) {
            if (live) bsum[(int64_t)b * r.n_list + pos] = acc;
            acc = 0.f;
        } else if (r.sum_mode == FT_SUM_BLOCKED) {
            tot += (double)acc;
            acc = 0.f;
        }
    }
    if (!SPLIT && live) r.stats[t] = (float)(tot + (double)acc);
}

__device__ __forceinline__ uint64_t ordered_bits(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return u >> 63 ? ~u : u | 1ull << 63;
}

__global__ __launch_bounds__(64) void list_check_init_kernel(ListCheck *res)
{
    uint64_t *q = (uint64_t *)res;
    if (threadIdx.x < sizeof(ListCheck) / 8) q[threadIdx.x] = threadIdx.x == 1 || threadIdx.x == 3 ? 0ull : ~0ull;
}

// Every array is read once; a workgroup's extremes are joined by one atomic each.
__global__ __launch_bounds__(256) void list_check_kernel(const double *f0, const double *f1, const double *sky, int64_t n,
                                                         double dt_lo, double dt_hi, ListCheck *res)
{
    __shared__ uint64_t sh[4][8];
    uint64_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = q == 1 || q == 3 ? 0ull : ~0ull;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)gridDim.x * 256) {
        const double a = f0[t], b = f1[t], x = sky[3 * t], y = sky[3 * t + 1], z = sky[3 * t + 2];
        const uint64_t ua = ordered_bits(a), ub = ordered_bits(b);
        v[0] = min(v[0], ua);
        v[1] = max(v[1], ua);
        v[2] = min(v[2], ub);
        v[3] = max(v[3], ub);
        if (!__builtin_isfinite(a) || !(a > 0.0)) v[4] = min(v[4], (uint64_t)t);
        if (!__builtin_isfinite(b)) v[5] = min(v[5], (uint64_t)t);
        if (!__builtin_isfinite(x) || !__builtin_isfinite(y) || !__builtin_isfinite(z)) v[6] = min(v[6], 2 * (uint64_t)t);
        else if (fabs(sqrt(x * x + y * y + z * z) - 1.0) > 1e-12) v[6] = min(v[6], 2 * (uint64_t)t + 1);
        if (!(a + fmin(b * dt_lo, b * dt_hi) > 0.0)) v[7] = min(v[7], (uint64_t)t);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint64_t y = __shfl_xor(v[q], o, 64);
            v[q] = q == 1 || q == 3 ? max(v[q], y) : min(v[q], y);
        }
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        const int q = threadIdx.x;
        const bool most = q == 1 || q == 3;
        uint64_t x = sh[0][q];
        for (int w = 1; w < 4; ++w) x = most ? max(x, sh[w][q]) : min(x, sh[w][q]);
        unsigned long long *at = (unsigned long long *)res + q;
        if (most) atomicMax(at, (unsigned long long)x);
        else if (x != ~0ull) atomicMin(at, (unsigned long long)x);
    }
}

// Templates in the order of LIST_KEYS equal steps of f0 (any order within one):
// counts, their running sum, places.  A workgroup counts 4096 templates in LDS
// and adds or takes its share of a step with one atomic.
constexpr int LIST_KEYS = 4096;

__device__ __forceinline__ int list_key(const EvalRun &r, int64_t t, double f_lo, double scale)
{
    return min(max((int)((r.f0[t] - f_lo) * scale), 0), LIST_KEYS - 1);
}

template <bool PLACE>
__global__ __launch_bounds__(1024) void list_order_kernel(EvalRun r, double f_lo, double scale, uint32_t *cnt, int32_t *order)
{
    __shared__ uint32_t h[LIST_KEYS];
    for (int q = threadIdx.x; q < LIST_KEYS; q += 1024) h[q] = 0;
    __syncthreads();
    int key[4];
    uint32_t rank[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t t = (int64_t)blockIdx.x * 4096 + i * 1024 + threadIdx.x;
        key[i] = t < r.n_list ? list_key(r, t, f_lo, scale) : -1;
        if (key[i] >= 0) rank[i] = atomicAdd(&h[key[i]], 1u);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < LIST_KEYS; q += 1024)
        if (h[q]) {
            const uint32_t at = atomicAdd(&cnt[q], h[q]);
            if (PLACE) h[q] = at;
        }
    if (!PLACE) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (key[i] >= 0) order[h[key[i]] + rank[i]] = (int32_t)((int64_t)blockIdx.x * 4096 + i * 1024 + threadIdx.x);
}

// Counts to first places, in place.
__global__ __launch_bounds__(1024) void list_scan_kernel(uint32_t *cnt)
{
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t v[4], own = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = cnt[4 * tid + i];
        own += v[i];
    }
    uint32_t incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[tid >> 6] = incl;
    __syncthreads();
    uint32_t at = incl - own;
    for (int w = 0; w < tid >> 6; ++w) at += wsum[w];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        cnt[4 * tid + i] = at;
        at += v[i];
    }
}

__global__ __launch_bounds__(1024) void list_clear_kernel(uint32_t *cnt) { cnt[blockIdx.x * 1024 + threadIdx.x] = 0; }

// Per-SFT parameters (s, v - v0) of the segments in mask, and s alone.
__global__ __launch_bounds__(256) void bank_par_kernel(const double *dt, const double *v, const uint32_t *mask,
                                                       int n_sft, double inv_hs, f32x4 *par, float *sval)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (n_sft + SUM_BLOCK - 1) / SUM_BLOCK * SUM_BLOCK) return;
    if (k >= n_sft) {
        sval[k] = 0.f;
        return;
    }
    const int b = k / SUM_BLOCK, j = k % SUM_BLOCK;
    const int len = min(SUM_BLOCK, n_sft - b * SUM_BLOCK);
    const uint32_t m = mask[b];
    const uint32_t upto = j == 31 ? m : m & ((2u << j) - 1u), after = m & ~upto;
    const int f = 31 - __builtin_clz(upto), l = after ? __builtin_ctz(after) - 1 : len - 1;
    const int kf = b * SUM_BLOCK + f, kl = b * SUM_BLOCK + l;
    const double *vk = v + 3 * (int64_t)k, *v0 = v + 3 * (int64_t)((kf + kl) >> 1);
    f32x4 q;
    q[0] = (float)((dt[k] - 0.5 * (dt[kf] + dt[kl])) * inv_hs);
    q[1] = (float)(vk[0] - v0[0]);
    q[2] = (float)(vk[1] - v0[1]);
    q[3] = (float)(vk[2] - v0[2]);
    par[k] = q;
    sval[k] = q[0];
}

// Velocity polynomial of one block per workgroup (64 lanes): least squares in
// the Chebyshev basis T_0 .. T_5 of s by the normal equations (well conditioned
// there), solved in FP64 by Cholesky, converted to powers of s and rounded to
// FP32 beyond the linear one; then the largest residual over the block's SFTs
// with those rounded coefficients.  The fit holds when the residual is at most
// res_max, the linear coefficient at most 2 max|v - v0| and the others' sum at
// most max|v - v0| (X and Y of the bound).
__global__ __launch_bounds__(64) void bank_fit_kernel(const double *v, const uint32_t *mask, const f32x4 *par, int n_sft,
                                                      double dv_max, double res_max, BankFit *fit)
{
    constexpr int D = 6;
    __shared__ double T[SUM_BLOCK][D], dv[SUM_BLOCK][3], G[D][D], rhs[D][3], mono[D][3];
    const int b = blockIdx.x, lane = threadIdx.x, k0 = b * SUM_BLOCK;
    if (mask[b] != 1u || n_sft - k0 < SUM_BLOCK) {
        if (lane == 0) fit[b].res = -1.f;
        return;
    }
    const double *v0 = v + 3 * (int64_t)((2 * k0 + SUM_BLOCK - 1) >> 1);
    if (lane < SUM_BLOCK) {
        const double s = (double)par[k0 + lane][0];
        T[lane][0] = 1.0;
        T[lane][1] = s;
        for (int j = 2; j < D; ++j) T[lane][j] = 2.0 * s * T[lane][j - 1] - T[lane][j - 2];
        for (int d = 0; d < 3; ++d) dv[lane][d] = v[3 * (int64_t)(k0 + lane) + d] - v0[d];
    }
    __syncthreads();
    if (lane < D * D) {
        double g = 0.0;
        for (int q = 0; q < SUM_BLOCK; ++q) g = fma(T[q][lane / D], T[q][lane % D], g);
        G[lane / D][lane % D] = g;
    } else if (lane < D * D + 3 * D) {
        const int i = (lane - D * D) / 3, d = (lane - D * D) % 3;
        double g = 0.0;
        for (int q = 0; q < SUM_BLOCK; ++q) g = fma(T[q][i], dv[q][d], g);
        rhs[i][d] = g;
    }
    __syncthreads();
    if (lane < 3) {  // one component a lane, the factorisation repeated
        double L[D][D], c[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            double x = G[j][j];
#pragma unroll
            for (int q = 0; q < j; ++q) x -= L[j][q] * L[j][q];
            L[j][j] = 1.0 / sqrt(x);  // the inverse of the diagonal
#pragma unroll
            for (int i = j + 1; i < D; ++i) {
                double y = G[i][j];
#pragma unroll
                for (int q = 0; q < j; ++q) y -= L[i][q] * L[j][q];
                L[i][j] = y * L[j][j];
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i) {
            double y = rhs[i][lane];
#pragma unroll
            for (int q = 0; q < i; ++q) y -= L[i][q] * c[q];
            c[i] = y * L[i][i];
        }
#pragma unroll
        for (int i = D - 1; i >= 0; --i) {
            double y = c[i];
#pragma unroll
            for (int q = i + 1; q < D; ++q) y -= L[q][i] * c[q];
            c[i] = y * L[i][i];
        }
        mono[0][lane] = c[0] - c[2] + c[4];
        mono[1][lane] = c[1] - 3.0 * c[3] + 5.0 * c[5];
        mono[2][lane] = 2.0 * c[2] - 8.0 * c[4];
        mono[3][lane] = 4.0 * c[3] - 20.0 * c[5];
        mono[4][lane] = 8.0 * c[4];
        mono[5][lane] = 16.0 * c[5];
        fit[b].v0[lane] = v0[lane] + mono[0][lane];
        fit[b].v1[lane] = mono[1][lane];
        for (int j = 2; j < D; ++j) fit[b].v[j - 2][lane] = (float)mono[j][lane];
    }
    __syncthreads();
    double r2 = 0.0, sum = 0.0;
    if (lane < SUM_BLOCK) {
        const double s = T[lane][1];
        for (int d = 0; d < 3; ++d) {
            double y = 0.0;
            for (int j = D - 1; j >= 2; --j) y = fma(s, y, (double)(float)mono[j][d]);
            y = fma(s, fma(s, y, mono[1][d]), mono[0][d]) - dv[lane][d];
            r2 = fma(y, y, r2);
        }
    }
    double lin = 0.0;
    for (int j = 1; j < D; ++j) {
        const double y = sqrt(mono[j][0] * mono[j][0] + mono[j][1] * mono[j][1] + mono[j][2] * mono[j][2]);
        if (j == 1) lin = y;
        else sum += y;
    }
    for (int o = 32; o > 0; o >>= 1) r2 = fmax(r2, __shfl_xor(r2, o, 64));
    const double res = sqrt(r2) * (1.0 + 1e-6) + 1e-18;
    if (lane == 0) {
        const bool ok = res <= res_max && lin <= 2.0 * dv_max && sum <= dv_max;  // false for a NaN
        fit[b].res = ok ? (float)(1.2500001 * res) : -1.f;
    }
}

template <int W>
hipError_t launch_w(const EvalRun &r, const BankPlan &pl, float *bsum, int bps, dim3 grid, hipStream_t s)
{
    const size_t lds = (size_t)2 * kBufFloats<W> * sizeof(float);
    if (bsum)
        hipLaunchKernelGGL((eval_bank_kernel<W, true>), grid, dim3(BANK_THREADS), lds, s, r, pl, bsum, bps);
    else
        hipLaunchKernelGGL((eval_bank_kernel<W, false>), grid, dim3(BANK_THREADS), lds, s, r, pl, bsum, bps);
    return hipGetLastError();
}

}  // namespace

size_t bank_fit_bytes(int n_blk) { return (size_t)n_blk * sizeof(BankFit); }

hipError_t launch_bank_tables(const EvalRun &run, const BankPlan &pl, double res_max, hipStream_t s)
{
    static_assert(SUM_BLOCK == 32, "one mask word per block");
    const int n_blk = (run.n_sft + SUM_BLOCK - 1) / SUM_BLOCK;
    hipLaunchKernelGGL(bank_par_kernel, dim3((unsigned)((n_blk + 7) / 8)), dim3(256), 0, s, run.dt, run.v, pl.mask,
                       run.n_sft, 1.0 / pl.hs, (f32x4 *)pl.par, pl.sval);
    hipLaunchKernelGGL(bank_fit_kernel, dim3((unsigned)n_blk), dim3(64), 0, s, run.v, pl.mask, (const f32x4 *)pl.par,
                       run.n_sft, pl.dv_max, res_max, (BankFit *)pl.fit);
    return hipGetLastError();
}

hipError_t launch_eval_bank(const EvalRun &run, const BankPlan &pl, float *bsum, int n_seg, hipStream_t s)
{
    if (run.n_list <= 0) return hipSuccess;
    const int n_blk = (run.n_sft + SUM_BLOCK - 1) / SUM_BLOCK;
    const int bps = bsum ? (n_blk + n_seg - 1) / n_seg : n_blk;
    const dim3 grid((unsigned)((run.n_list + BANK_THREADS - 1) / BANK_THREADS), bsum ? (unsigned)((n_blk + bps - 1) / bps) : 1u);
    hipError_t e = pl.width <= 128   ? launch_w<128>(run, pl, bsum, bps, grid, s)
                   : pl.width <= 256 ? launch_w<256>(run, pl, bsum, bps, grid, s)
                   : pl.width <= BANK_MAX_WIDTH
                       ? launch_w<512>(run, pl, bsum, bps, grid, s)
                       : hipErrorInvalidValue;
    if (e == hipSuccess && bsum)
        e = launch_block_sum(bsum, run.n_list, n_blk, run.stats, nullptr, s);
    return e;
}

hipError_t launch_list_check(const double *f0, const double *f1, const double *sky, int64_t n, double dt_lo, double dt_hi,
                             ListCheck *res, hipStream_t s)
{
    hipLaunchKernelGGL(list_check_init_kernel, dim3(1), dim3(64), 0, s, res);
    const unsigned g = (unsigned)((n + 255) / 256 < 512 ? (n + 255) / 256 : 512);
    hipLaunchKernelGGL(list_check_kernel, dim3(g), dim3(256), 0, s, f0, f1, sky, n, dt_lo, dt_hi, res);
    return hipGetLastError();
}

size_t list_order_keys() { return LIST_KEYS; }

hipError_t launch_list_window(const EvalRun &run, const BankPlan &pl, const ListPlan &lp, float *bsum, int n_seg, hipStream_t s)
{
    if (run.n_list <= 0) return hipSuccess;
    const int n_blk = (run.n_sft + SUM_BLOCK - 1) / SUM_BLOCK;
    const int bps = bsum ? (n_blk + n_seg - 1) / n_seg : n_blk;
    const double scale = lp.f0_hi > lp.f0_lo ? LIST_KEYS / (lp.f0_hi - lp.f0_lo) : 0.0;
    const dim3 go((unsigned)((run.n_list + 4095) / 4096));
    hipLaunchKernelGGL(list_clear_kernel, dim3(LIST_KEYS / 1024), dim3(1024), 0, s, lp.cnt);
    hipLaunchKernelGGL(list_order_kernel<false>, go, dim3(1024), 0, s, run, lp.f0_lo, scale, lp.cnt, lp.order);
    hipLaunchKernelGGL(list_scan_kernel, dim3(1), dim3(1024), 0, s, lp.cnt);
    hipLaunchKernelGGL(list_order_kernel<true>, go, dim3(1024), 0, s, run, lp.f0_lo, scale, lp.cnt, lp.order);
    const dim3 grid((unsigned)((run.n_list + BANK_THREADS - 1) / BANK_THREADS), bsum ? (unsigned)((n_blk + bps - 1) / bps) : 1u);
    const size_t lds = (size_t)2 * kListFloats * sizeof(float);
    if (bsum)
        hipLaunchKernelGGL(eval_list_kernel<true>, grid, dim3(BANK_THREADS), lds, s, run, pl, lp.order, lp.dt_lo, lp.dt_hi, bsum, bps);
    else
        hipLaunchKernelGGL(eval_list_kernel<false>, grid, dim3(BANK_THREADS), lds, s, run, pl, lp.order, lp.dt_lo, lp.dt_hi, bsum, bps);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && bsum) e = launch_block_sum(bsum, run.n_list, n_blk, run.stats, lp.order, s);
    return e;
}

}  // namespace ft
