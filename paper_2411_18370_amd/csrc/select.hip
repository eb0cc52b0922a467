// Exact per-sub-band toplists (the list of loudest candidates per region of
// Secs. IV.B and VI) from the FP32 statistic.
//
// 1. Radix select (4 passes of 8-bit digits over the IEEE bits of S32, which
//    order like the values since S32 >= 0) finds K32, the exact K-th largest
//    FP32 statistic of each sub-band.
// 2. Every template with S32 >= K32 (1 - 2e)/(1 + 2e) is a candidate, where e
//    bounds |S32 - S64| / S relative to the sum: if K templates have
//    S32 >= K32 then the K-th largest S64 is >= K32/(1 + e), so every member of
//    the FP64 top-K has S32 >= K32 (1 - e)/(1 + e).  Candidates are compacted
//    per sub-band.
// 3. Each candidate is re-summed in FP64 in SFT order with canonical bins
//    (a workgroup per candidate: three wavefronts form the weighted terms and
//    store them to LDS; the fourth adds them to the running sum, 256 at a time
//    with the bits of the plain sequential FP64 sum).
// 4. Candidates are ranked within their sub-band by (S64 desc, index asc);
//    ranks < K are the toplist, identical to sorting all FP64 statistics.
#include "ft_internal.h"

#include <algorithm>

namespace ft {

namespace {

constexpr uint32_t NAN_KEY = 0x7f800000u;  // keys above this are NaN
constexpr int ST = 8;                      // state words per segment
enum { S_PREFIX = 0, S_MASK = 1, S_KREM = 2, S_DONE = 3, S_THR = 4 };

// Prepares an evaluation's selection: clears the error flags, maps the f0
// values to sub-bands (n = 0: no mapping) and sets the selection's counters.
__global__ __launch_bounds__(256) void select_prep_kernel(const double *f0, int64_t n, const double *edges, int n_sub,
                                                          int32_t *seg, int k, SelectBufs b, uint32_t *err)
{
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (i0 == 0) *err = 0u;
    for (int64_t q = i0; q < SEL_TICKETS; q += step) b.ticket[q] = 0u;
    for (int64_t q = i0; q < (int64_t)4 * n_sub * 256; q += step) b.hist[q] = 0u;
    for (int64_t sg = i0; sg < n_sub; sg += step) {
        uint32_t *st = b.state + sg * ST;
        st[S_PREFIX] = 0;
        st[S_MASK] = 0;
        st[S_KREM] = (uint32_t)k;
        st[S_DONE] = 0;
        st[S_THR] = 0;
        b.cnt[sg] = 0;
        b.fill[sg] = 0;
    }
    for (int64_t q = i0; q < n; q += step) {
        const double f = f0[q];
        int lo = 0, hi = n_sub;  // find the last edge <= f
        if (!(edges[0] <= f) || !(f < edges[n_sub])) {
            seg[q] = -1;
            continue;
        }
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (edges[mid] <= f) lo = mid;
            else hi = mid;
        }
        seg[q] = lo;
    }
}

// True in every thread of the grid's last workgroup to get here.  What the
// workgroups hand over are device-scope atomics alone (histograms and counts),
// read back by device-scope loads: each wave waits until its own have been
// performed, then the ticket orders the workgroups.  A device fence would also
// write back and drop caches, once a workgroup: measured 70 us a pass over 2048
// of them.  Workgroups take tickets in SEL_GROUPS groups, each on a cache line
// of its own, and the last of each group takes one of the pass: atomics on one
// address are performed one by one (about 10 ns each).
__device__ __forceinline__ bool last_block(uint32_t *ticket)
{
    __shared__ uint32_t last;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t n = gridDim.x, g = blockIdx.x % SEL_GROUPS, members = (n - g + SEL_GROUPS - 1) / SEL_GROUPS;
        last = 0;
        if (__hip_atomic_fetch_add(ticket + (1 + g) * SEL_LINE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1)
            last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   min(n, (uint32_t)SEL_GROUPS) - 1;
    }
    __syncthreads();
    return last;
}

// One wave chooses the digit holding the k_rem-th largest key of a segment from
// its histogram h(d): lane l sums digits 255 - 4 l .. 252 - 4 l, a scan over the
// lanes finds the four that hold it.  Updates the segment's state (every lane
// calls it and reads the state; the lane that finds the digit writes it).
template <typename H>
__device__ __forceinline__ void choose_digit(H h, uint32_t *st, int shift, double two_e)
{
    const int lane = threadIdx.x & 63;
    const uint32_t done = st[S_DONE], k_rem = st[S_KREM], prefix = st[S_PREFIX], mask = st[S_MASK];
    if (done) return;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = h(255 - 4 * lane - i);
        sum += v[i];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    const uint64_t reach = __builtin_amdgcn_ballot_w64(incl >= k_rem);
    if (reach == 0) {  // fewer than K members: all of them are candidates
        if (lane == 0) {
            st[S_DONE] = 1;
            st[S_THR] = 0;
        }
        return;
    }
    if (lane != __builtin_ctzll(reach)) return;
    uint32_t cum = incl - sum;
    int found = 255 - 4 * lane;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if (cum + v[i] >= k_rem) break;
        cum += v[i];
        --found;
    }
    const uint32_t key = prefix | (uint32_t)found << shift;
    st[S_PREFIX] = key;
    st[S_MASK] = mask | 255u << shift;
    st[S_KREM] = k_rem - cum;
    if (shift == 0) {
        const double kth = (double)__uint_as_float(key);
        const double thr = kth * (1.0 - two_e) / (1.0 + two_e);
        float tf = (float)thr;
        if ((double)tf > thr) tf = nextafterf(tf, 0.f);
        if (!(tf > 0.f)) tf = 0.f;
        st[S_THR] = __float_as_uint(tf);
        st[S_DONE] = 1;
    }
}

// End of a histogram pass in LDS (at most 32 sub-bands): the last workgroup
// chooses every segment's digit.
__device__ __forceinline__ void hist_done(uint32_t *state, const uint32_t *hist, int n_seg, int shift, double two_e,
                                          uint32_t *ticket)
{
    if (!last_block(ticket)) return;
    for (int sg = threadIdx.x >> 6; sg < n_seg; sg += blockDim.x >> 6) {
        const uint32_t *h = hist + (int64_t)sg * 256;
        choose_digit([&](int d) { return __hip_atomic_load(h + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                     state + (int64_t)sg * ST, shift, two_e);
    }
}

// End of the count: the last workgroup forms the segments' offsets in the
// candidate list and the toplist lengths.
__device__ __forceinline__ void count_done(const SelectBufs &b, int n_seg, int k, uint32_t *ticket, uint32_t *err)
{
    __shared__ uint64_t part[256];
    if (!last_block(ticket)) return;
    const int tid = threadIdx.x, per = (n_seg + 255) / 256;
    const int s0 = min(tid * per, n_seg), s1 = min(s0 + per, n_seg);
    auto cnt = [&](int sg) { return __hip_atomic_load(b.cnt + sg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    uint64_t own = 0;
    for (int sg = s0; sg < s1; ++sg) own += cnt(sg);
    part[tid] = own;
    __syncthreads();
    uint64_t acc = 0;
    for (int q = 0; q < tid; ++q) acc += part[q];
    if (tid == 0) b.off[0] = 0;
    for (int sg = s0; sg < s1; ++sg) {
        const uint32_t c = cnt(sg);
        acc += c;
        b.off[sg + 1] = (uint32_t)(acc < 0xffffffffull ? acc : 0xffffffffull);
        b.n_out[sg] = (int32_t)min(c, (uint32_t)k);
    }
    if (tid == 255 && acc > (uint64_t)b.cap) atomicOr(err, ERR_CAND_OVERFLOW);
}

// Iterate the templates of a bank as rows: GRID rows are (s, j) pairs of
// n_f0 templates whose sub-band depends on i only; LIST rows are chunks.
struct Rows {
    int64_t n_rows, row_len, n_total;
    bool grid;
};

__device__ __forceinline__ int seg_at(const int32_t *seg_of, const Rows &rw, int64_t c,
                                      int64_t t)
{
    return rw.grid ? seg_of[c] : seg_of[t];
}

template <bool LDS>
__global__ __launch_bounds__(256) void hist_kernel(const float *stats, const int32_t *seg_of,
                                                   Rows rw, uint32_t *state, uint32_t *hist, int n_seg,
                                                   int shift, double two_e, uint32_t *ticket)
{
    extern __shared__ uint32_t hsh[];
    if (LDS) {
        for (int q = threadIdx.x; q < n_seg * 256; q += blockDim.x) hsh[q] = 0;
        __syncthreads();
    }
    for (int64_t row = blockIdx.x; row < rw.n_rows; row += gridDim.x) {
        for (int64_t c = threadIdx.x; c < rw.row_len; c += blockDim.x) {
            const int64_t t = row * rw.row_len + c;
            if (t >= rw.n_total) break;
            const int sg = seg_at(seg_of, rw, c, t);
            if (sg < 0) continue;
            const uint32_t *st = state + (int64_t)sg * ST;
            if (st[S_DONE]) continue;
            const uint32_t key = __float_as_uint(stats[t]);
            if (key > NAN_KEY || (key & st[S_MASK]) != st[S_PREFIX]) continue;
            const uint32_t digit = (key >> shift) & 255u;
            if (LDS) atomicAdd(&hsh[sg * 256 + digit], 1u);
            else atomicAdd(&hist[(int64_t)sg * 256 + digit], 1u);
        }
    }
    if (LDS) {
        __syncthreads();
        for (int q = threadIdx.x; q < n_seg * 256; q += blockDim.x)
            if (hsh[q]) atomicAdd(&hist[q], hsh[q]);
    }
    if (LDS) hist_done(state, hist, n_seg, shift, two_e, ticket);
}

// The digits after a histogram pass without LDS (more than 32 sub-bands), a wave
// each: the pass's last workgroup alone took 0.8 ms a pass for 4096 sub-bands,
// a thread each 37 us, this 6 us.
__global__ __launch_bounds__(256) void digits_kernel(uint32_t *state, const uint32_t *hist, int n_seg, int shift, double two_e)
{
    const int sg = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (sg >= n_seg) return;
    const uint32_t *h = hist + (int64_t)sg * 256;
    choose_digit([&](int d) { return h[d]; }, state + (int64_t)sg * ST, shift, two_e);
}

// Grid banks: a row is one (sky, f1) pair of n_f0 templates and the sub-band
// depends on the f0 column only, so each thread owns the columns
// threadIdx.x + 256 i (i < COLS) of every row it visits and keeps their
// sub-band and selection state in registers; the rows stream through.
template <int COLS>
struct GridCols {
    int32_t sg[COLS];
    bool on[COLS];
};

template <int COLS>
__device__ __forceinline__ GridCols<COLS> grid_cols(const int32_t *seg_of, const Rows &rw)
{
    GridCols<COLS> g;
#pragma unroll
    for (int i = 0; i < COLS; ++i) {
        const int64_t c = threadIdx.x + 256 * i;
        g.sg[i] = c < rw.row_len ? seg_of[c] : -1;
        g.on[i] = g.sg[i] >= 0;
    }
    return g;
}

// Histogram pass over grid rows.  When every lane of the wave with a key for
// this column hits the same (sub-band, digit) -- the common case in the first
// passes, where a row's statistics share their leading bits -- one lane adds
// the wave's count.
template <int COLS>
__global__ __launch_bounds__(256) void hist_grid_kernel(const float *stats, const int32_t *seg_of, Rows rw,
                                                        uint32_t *state, uint32_t *hist, int n_seg, int shift,
                                                        double two_e, uint32_t *ticket)
{
    extern __shared__ uint32_t hsh[];
    for (int q = threadIdx.x; q < n_seg * 256; q += blockDim.x) hsh[q] = 0;
    GridCols<COLS> g = grid_cols<COLS>(seg_of, rw);
    uint32_t mask[COLS], prefix[COLS];
#pragma unroll
    for (int i = 0; i < COLS; ++i) {
        const uint32_t *st = state + (int64_t)max(g.sg[i], 0) * ST;
        g.on[i] = g.on[i] && !st[S_DONE];
        mask[i] = st[S_MASK];
        prefix[i] = st[S_PREFIX];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int64_t row = blockIdx.x; row < rw.n_rows; row += gridDim.x) {
        const float *rp = stats + row * rw.row_len;
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
            int idx = -1;
            if (g.on[i]) {
                const uint32_t key = __float_as_uint(rp[threadIdx.x + 256 * i]);
                if (key <= NAN_KEY && (key & mask[i]) == prefix[i]) idx = g.sg[i] * 256 + (int)((key >> shift) & 255u);
            }
            const uint64_t valid = __builtin_amdgcn_ballot_w64(idx >= 0);
            if (valid == 0) continue;
            const int first = __builtin_ctzll(valid);
            const int lead = __builtin_amdgcn_readlane(idx, first);
            const uint64_t same = __builtin_amdgcn_ballot_w64(idx == lead);
            if (same == valid) {
                if (lane == first) atomicAdd(&hsh[lead], (uint32_t)__builtin_popcountll(valid));
            } else if (idx >= 0) {
                atomicAdd(&hsh[idx], 1u);
            }
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < n_seg * 256; q += blockDim.x)
        if (hsh[q]) atomicAdd(&hist[q], hsh[q]);
    hist_done(state, hist, n_seg, shift, two_e, ticket);
}

// Candidates per sub-band over grid rows: counts kept per column in
// registers, added once per thread.
template <int COLS>
__global__ __launch_bounds__(256) void count_grid_kernel(const float *stats, const int32_t *seg_of, Rows rw,
                                                         const uint32_t *state, SelectBufs b, int n_seg, int k,
                                                         uint32_t *err)
{
    extern __shared__ uint32_t csh[];
    for (int q = threadIdx.x; q < n_seg; q += blockDim.x) csh[q] = 0;
    GridCols<COLS> g = grid_cols<COLS>(seg_of, rw);
    uint32_t thr[COLS], n[COLS];
#pragma unroll
    for (int i = 0; i < COLS; ++i) {
        thr[i] = state[(int64_t)max(g.sg[i], 0) * ST + S_THR];
        n[i] = 0;
    }
    __syncthreads();
    for (int64_t row = blockIdx.x; row < rw.n_rows; row += gridDim.x) {
        const float *rp = stats + row * rw.row_len;
#pragma unroll
        for (int i = 0; i < COLS; ++i)
            if (g.on[i]) {
                const uint32_t key = __float_as_uint(rp[threadIdx.x + 256 * i]);
                n[i] += (key <= NAN_KEY && key >= thr[i]) ? 1u : 0u;
            }
    }
#pragma unroll
    for (int i = 0; i < COLS; ++i)
        if (g.on[i] && n[i]) atomicAdd(&csh[g.sg[i]], n[i]);
    __syncthreads();
    for (int q = threadIdx.x; q < n_seg; q += blockDim.x)
        if (csh[q]) atomicAdd(&b.cnt[q], csh[q]);
    count_done(b, n_seg, k, b.ticket + 4 * SEL_TICKET, err);
}

// Compaction of the candidates over grid rows.
template <int COLS>
__global__ __launch_bounds__(256) void scatter_grid_kernel(const float *stats, const int32_t *seg_of, Rows rw,
                                                           const uint32_t *state, const uint32_t *off,
                                                           uint32_t *fill, int64_t *cand, int64_t cap)
{
    GridCols<COLS> g = grid_cols<COLS>(seg_of, rw);
    uint32_t thr[COLS];
#pragma unroll
    for (int i = 0; i < COLS; ++i) thr[i] = state[(int64_t)max(g.sg[i], 0) * ST + S_THR];
    for (int64_t row = blockIdx.x; row < rw.n_rows; row += gridDim.x) {
        const float *rp = stats + row * rw.row_len;
#pragma unroll
        for (int i = 0; i < COLS; ++i)
            if (g.on[i]) {
                const int64_t c = threadIdx.x + 256 * i;
                const uint32_t key = __float_as_uint(rp[c]);
                if (key <= NAN_KEY && key >= thr[i]) {
                    const int64_t pos = (int64_t)off[g.sg[i]] + atomicAdd(&fill[g.sg[i]], 1u);
                    if (pos < cap) cand[pos] = row * rw.row_len + c;
                }
            }
    }
}

__global__ __launch_bounds__(256) void count_kernel(const float *stats, const int32_t *seg_of,
                                                    Rows rw, const uint32_t *state, SelectBufs b, int n_seg,
                                                    int k, uint32_t *err)
{
    extern __shared__ uint32_t csh[];
    for (int q = threadIdx.x; q < n_seg; q += blockDim.x) csh[q] = 0;
    __syncthreads();
    for (int64_t row = blockIdx.x; row < rw.n_rows; row += gridDim.x) {
        for (int64_t c = threadIdx.x; c < rw.row_len; c += blockDim.x) {
            const int64_t t = row * rw.row_len + c;
            if (t >= rw.n_total) break;
            const int sg = seg_at(seg_of, rw, c, t);
            if (sg < 0) continue;
            const uint32_t key = __float_as_uint(stats[t]);
            if (key > NAN_KEY || key < state[(int64_t)sg * ST + S_THR]) continue;
            atomicAdd(&csh[sg], 1u);
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < n_seg; q += blockDim.x)
        if (csh[q]) atomicAdd(&b.cnt[q], csh[q]);
    count_done(b, n_seg, k, b.ticket + 4 * SEL_TICKET, err);
}

__global__ __launch_bounds__(256) void scatter_kernel(const float *stats, const int32_t *seg_of,
                                                      Rows rw, const uint32_t *state,
                                                      const uint32_t *off, uint32_t *fill,
                                                      int64_t *cand, int64_t cap)
{
    for (int64_t row = blockIdx.x; row < rw.n_rows; row += gridDim.x) {
        for (int64_t c = threadIdx.x; c < rw.row_len; c += blockDim.x) {
            const int64_t t = row * rw.row_len + c;
            if (t >= rw.n_total) break;
            const int sg = seg_at(seg_of, rw, c, t);
            if (sg < 0) continue;
            const uint32_t key = __float_as_uint(stats[t]);
            if (key > NAN_KEY || key < state[(int64_t)sg * ST + S_THR]) continue;
            const int64_t pos = (int64_t)off[sg] + atomicAdd(&fill[sg], 1u);
            if (pos < cap) cand[pos] = t;
        }
    }
}

struct TemplateParams {
    double f0, f1, nx, ny, nz;
    double aw, omega, phib;  // binary-system list banks (aw = a_p Omega), else 0
};

__device__ __forceinline__ TemplateParams params_of(const EvalRun &r, bool grid, int64_t t)
{
    TemplateParams p;
    int64_t s;
    if (grid) {
        const int64_t i = t % r.n_f0;
        const int64_t rest = t / r.n_f0;
        const int64_t j = rest % r.n_f1;
        s = rest / r.n_f1;
        p.f0 = r.f0[i];
        p.f1 = r.f1[j];
    } else {
        s = t;
        p.f0 = r.f0[t];
        p.f1 = r.ap ? 0.0 : r.f1[t];
    }
    p.aw = p.omega = p.phib = 0.0;
    if (!grid && r.ap) {
        p.omega = r.omega[t];
        p.phib = r.phib[t];
        p.aw = r.ap[t] * p.omega;
    }
    p.nx = r.sky[3 * s];
    p.ny = r.sky[3 * s + 1];
    p.nz = r.sky[3 * s + 2];
    return p;
}

// Table values at the canonical bins of a template at SFTs k + 64 j, j < 4 (past
// the last SFT: the last one's) and their weights: u_k, with sky-dependent
// weights times ab_k(n) inv, inv = 1 / sum_k' u_k' ab_k'(n).  Four at a time
// without a branch between them, so their loads are in flight together.
__device__ __forceinline__ void rescore_terms(const EvalRun &r, const TemplateParams &tp, int k0, bool sky, double inv,
                                              uint32_t &bad, float (&p)[4], double (&w)[4])
{
    double vx[4], vy[4], vz[4], dt[4];
    int b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = min(k0 + 64 * j, r.n_sft - 1);
        const double *vk = r.v + 3 * (int64_t)k;
        vx[j] = vk[0];
        vy[j] = vk[1];
        vz[j] = vk[2];
        dt[j] = r.dt[k];
        w[j] = 1.0;
    }
    if (r.weight) {
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = (double)r.weight[min(k0 + 64 * j, r.n_sft - 1)];
    }
    if (r.ap) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            b[j] = bin_binary(tp.f0, doppler_factor(vx[j], vy[j], vz[j], tp.nx, tp.ny, tp.nz), tp.aw, tp.omega, tp.phib,
                              dt[j], r.t_sft);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            b[j] = bin_fp64(tp.f0, tp.f1 * dt[j], doppler_factor(vx[j], vy[j], vz[j], tp.nx, tp.ny, tp.nz), r.t_sft);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = min(k0 + 64 * j, r.n_sft - 1);
        const int c = min(max(b[j] - r.first_bin, 0), r.n_bins - 1);
        bad |= c != b[j] - r.first_bin ? ERR_RANGE : 0u;
        p[j] = r.power[(int64_t)k * r.n_bins + c];
    }
    if (sky) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            w[j] = w[j] * (sky_ab(r.arms + 6 * (int64_t)min(k0 + 64 * j, r.n_sft - 1), tp.nx, tp.ny, tp.nz) * inv);
    }
}

// Sequential FP64 sums over the SFTs, a group of NW waves per template: waves
// 1 .. NW-1 of the group form the terms of a chunk of 256 (NW - 1) SFTs into one
// of two LDS buffers while wave 0 adds an earlier chunk in SFT order (the same
// bits as term by term).  terms(k, p, w) gives the table values of SFTs k + 64 j,
// j < 4 (loads in flight until the next chunk's bins are formed; anything past
// the last SFT) and their weights; acc = sum w p, and
// with MOM sw = sum w, sw2 = sum w^2 (the results are wave 0 lane 0's).
// What binds it are the terms' dependent gathers, hidden one chunk deep; added
// term by term by one lane, 10^4 additions took 57 us, 33 us as wave_chain does
// them.  Called by every thread of the workgroup with the same n_sft (the
// groups share its barriers); a group without a template is inactive.
constexpr int SEQ_PER_WAVE = 256;
template <int NW, bool MOM>
struct SeqBuf {
    static constexpr int CH = (NW - 1) * SEQ_PER_WAVE;
    double val[2][CH];
    double w[MOM ? 2 : 1][MOM ? CH : 1];
};

template <int NW, bool MOM, typename F>
__device__ __forceinline__ void seq_sums(F terms, int n_sft, SeqBuf<NW, MOM> &buf, int wave, bool active, double &acc,
                                         double &sw, double &sw2)
{
    constexpr int CH = SeqBuf<NW, MOM>::CH;
    const int lane = threadIdx.x & 63;
    const int n_ch = (n_sft + CH - 1) / CH;
    acc = sw = sw2 = 0.0;
    if (wave == 0) __builtin_amdgcn_s_setprio(3);  // the chain goes first on its SIMD
    float p[4] = {0.f, 0.f, 0.f, 0.f};
    double w[4] = {0.0, 0.0, 0.0, 0.0};
    // iteration it: the terms of chunk it are formed, those of chunk it - 1 go
    // to LDS, chunk it - 2 is added
    for (int it = 0; it <= n_ch + 1; ++it) {
        if (!active) {
        } else if (wave > 0) {
            const int q0 = (wave - 1) * SEQ_PER_WAVE + lane;
            float pn[4] = {0.f, 0.f, 0.f, 0.f};
            double wn[4] = {0.0, 0.0, 0.0, 0.0};
            if (it < n_ch) terms(it * CH + q0, pn, wn);
            if (it > 0 && it <= n_ch) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    buf.val[(it - 1) & 1][q0 + 64 * j] = w[j] * (double)p[j];
                    if (MOM) buf.w[(it - 1) & 1][q0 + 64 * j] = w[j];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                p[j] = pn[j];
                w[j] = wn[j];
            }
        } else if (it > 1) {
            const double *x = buf.val[it & 1], *y = buf.w[MOM ? it & 1 : 0];
            const int m = min(CH, n_sft - (it - 2) * CH);
            for (int q0 = 0; q0 < m; q0 += 256) {
                const int n = min(256, m - q0);
                acc = wave_chain(acc, [&](int q) { return x[q0 + q]; }, n);
                if (MOM) {
                    sw = wave_chain(sw, [&](int q) { return y[q0 + q]; }, n);
                    sw2 = wave_chain(sw2, [&](int q) { return y[q0 + q] * y[q0 + q]; }, n);
                }
            }
        }
        __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
}

// FP64 re-summation of template t in SFT order with canonical bins by one
// workgroup (seq_sums).  With MOM the weight sums W1 = sum w and W2 = sum w^2
// come out as well.  Four waves: three form 768 terms in about the time one
// adds them, and a chunk's rows stay in an XCD's L2 for the other candidates
// (eight waves: 238 against 134 us for the 1000 candidates of an all-sky band).
constexpr int RS_WAVES = 4;

template <bool MOM>
__device__ __forceinline__ double rescore_one(const EvalRun &r, bool grid, int64_t t, uint32_t &bad,
                                              SeqBuf<RS_WAVES, MOM> &buf, double *inv_sh, double &w1, double &w2)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const TemplateParams tp = params_of(r, grid, t);
    // sky-dependent weights: normalised per sky point (grid, precomputed) or per
    // template (binary banks, here)
    const bool bsky = !grid && r.arms;
    double inv = grid && r.sky_norm ? r.sky_norm[t / ((int64_t)r.n_f0 * r.n_f1)] : 0.0;
    if (bsky) {
        double c, d0, d1;
        seq_sums<RS_WAVES, MOM>(
            [&](int k0, float (&p)[4], double (&w)[4]) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = min(k0 + 64 * j, r.n_sft - 1);
                    p[j] = 1.f;
                    w[j] = (r.weight ? (double)r.weight[k] : 1.0) * sky_ab(r.arms + 6 * (int64_t)k, tp.nx, tp.ny, tp.nz);
                }
            },
            r.n_sft, buf, wave, true, c, d0, d1);
        if (threadIdx.x == 0) *inv_sh = 1.0 / c;
        __syncthreads();
        inv = *inv_sh;
    }
    double acc;
    seq_sums<RS_WAVES, MOM>(
        [&](int k, float (&p)[4], double (&w)[4]) {
            rescore_terms(r, tp, k, (grid && r.sky_norm) || bsky, inv, bad, p, w);
        },
        r.n_sft, buf, wave, true, acc, w1, w2);
    return acc;
}

// The same sum by one wavefront (per-SFT or per-sky-point weights): lanes form
// 256 terms at a time in the wave's LDS slice for wave_chain; the next terms'
// gathers are issued before the additions.  For candidates by the thousand:
// waves enough are in flight, and four per candidate only wait.
constexpr int RS_UNROLL = 4;

__device__ __forceinline__ double rescore_wave(const EvalRun &r, bool grid, int64_t t, int lane, uint32_t &bad,
                                               double *buf)
{
    const TemplateParams tp = params_of(r, grid, t);
    const bool sky = grid && r.sky_norm;
    const double inv = sky ? r.sky_norm[t / ((int64_t)r.n_f0 * r.n_f1)] : 0.0;
    float p[RS_UNROLL];
    double w[RS_UNROLL];
    double acc = 0.0;
    rescore_terms(r, tp, lane, sky, inv, bad, p, w);
    for (int k0 = 0; k0 < r.n_sft; k0 += 64 * RS_UNROLL) {
        double val[RS_UNROLL];
#pragma unroll
        for (int j = 0; j < RS_UNROLL; ++j) val[j] = w[j] * (double)p[j];
        if (k0 + 64 * RS_UNROLL < r.n_sft) rescore_terms(r, tp, k0 + 64 * RS_UNROLL + lane, sky, inv, bad, p, w);
#pragma unroll
        for (int j = 0; j < RS_UNROLL; ++j) buf[64 * j + lane] = val[j];
        wave_lds_sync();
        static_assert(64 * RS_UNROLL <= 256, "one step of wave_chain");
        acc = wave_chain(acc, [&](int q) { return buf[q]; }, min(64 * RS_UNROLL, r.n_sft - k0));
        wave_lds_sync();
    }
    return acc;
}

__global__ __launch_bounds__(256) void rescore_many_kernel(EvalRun r, bool grid, const int64_t *cand, const uint32_t *off,
                                                           int n_seg, int64_t cap, double *s64)
{
    __shared__ double rs_buf[4][64 * RS_UNROLL];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t total = min((int64_t)off[n_seg], cap);
    uint32_t bad = 0;
    for (int64_t p = (int64_t)blockIdx.x * 4 + wave; p < total; p += (int64_t)gridDim.x * 4) {
        const double acc = rescore_wave(r, grid, cand[p], lane, bad, rs_buf[wave]);
        if (lane == 0) s64[p] = acc;
    }
    if (bad) atomicOr(r.err, bad);
}

// FP64 re-summation of the candidates, one workgroup per candidate; with MOM,
// also each candidate's sums of weights and squared weights.
template <bool MOM>
__global__ __launch_bounds__(64 * RS_WAVES) void rescore_kernel(EvalRun r, bool grid, const int64_t *cand,
                                                                const uint32_t *off, int n_seg, int64_t cap, double *s64,
                                                                double *mom)
{
    __shared__ SeqBuf<RS_WAVES, MOM> buf;
    __shared__ double inv_sh;
    const int64_t total = min((int64_t)off[n_seg], cap);
    uint32_t bad = 0;
    for (int64_t p = blockIdx.x; p < total; p += gridDim.x) {
        double w1, w2;
        const double acc = rescore_one<MOM>(r, grid, cand[p], bad, buf, &inv_sh, w1, w2);
        if (threadIdx.x == 0) {
            s64[p] = acc;
            if (MOM) {
                mom[2 * p] = w1;
                mom[2 * p + 1] = w2;
            }
        }
    }
    if (bad) atomicOr(r.err, bad);
}

// FP64 re-summation of the templates of toplist entries top[0 .. n_out[0]):
// out[3p .. 3p+2] = (sum, W1, W2).
__global__ __launch_bounds__(64 * RS_WAVES) void rescore_entries_kernel(EvalRun r, bool grid, const ft_candidate *top,
                                                                        const int32_t *n_out, double *out)
{
    __shared__ SeqBuf<RS_WAVES, true> buf;
    __shared__ double inv_sh;
    const int64_t total = n_out[0];
    uint32_t bad = 0;
    for (int64_t p = blockIdx.x; p < total; p += gridDim.x) {
        double w1, w2;
        const double acc = rescore_one<true>(r, grid, top[p].index, bad, buf, &inv_sh, w1, w2);
        if (threadIdx.x == 0) {
            out[3 * p] = acc;
            out[3 * p + 1] = w1;
            out[3 * p + 2] = w2;
        }
    }
    if (bad) atomicOr(r.err, bad);
}

// Rank of each candidate within its sub-band under (S64 desc, index asc), one
// wave per candidate: 64 rivals are compared at a time, until k are ahead.
__global__ __launch_bounds__(256) void rank_kernel(EvalRun r, bool grid, const int64_t *cand,
                                                   const double *s64, const uint32_t *off,
                                                   int n_seg, int64_t cap, int k,
                                                   const double *mu_sigma, const double *mom,
                                                   ft_candidate *out)
{
    const int64_t total = min((int64_t)off[n_seg], cap);
    const int lane = threadIdx.x & 63;
    for (int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); p < total; p += (int64_t)gridDim.x * 4) {
        int lo = 0, hi = n_seg;  // segment: off[sg] <= p < off[sg+1]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((int64_t)off[mid] <= p) lo = mid;
            else hi = mid;
        }
        const int sg = lo;
        const int64_t q0 = off[sg];
        const int64_t q1 = min((int64_t)off[sg + 1], cap);
        const double sp = s64[p];
        const int64_t tp = cand[p];
        int64_t rank = 0;
        for (int64_t q = q0; q < q1 && rank < k; q += 64) {
            bool ahead = false;
            if (q + lane < q1) {
                const double sq = s64[q + lane];
                ahead = (sq > sp) || (sq == sp && cand[q + lane] < tp);
            }
            rank += __builtin_popcountll(__builtin_amdgcn_ballot_w64(ahead));
        }
        if (rank < k && lane == 0) {
            const TemplateParams par = params_of(r, grid, tp);
            ft_candidate c;
            c.index = tp;
            c.sub = sg;
            c.s32 = r.stats[tp];
            c.f0 = par.f0;
            c.f1 = par.f1;
            c.n[0] = par.nx;
            c.n[1] = par.ny;
            c.n[2] = par.nz;
            c.s64 = sp;
            // sky-dependent weights: the moments of the template's sky point
            // (grid) or of the template's own weights (binary banks)
            double own[2];
            const double *ms = mu_sigma;
            if (grid && r.sky_ms) {
                ms = r.sky_ms + 2 * (tp / ((int64_t)r.n_f0 * r.n_f1));
            } else if (mom) {
                stat_moments(r.stat, mom[2 * p], mom[2 * p + 1], own);
                ms = own;
            }
            c.z = (sp - ms[0]) / ms[1];
            out[(int64_t)sg * k + rank] = c;
        }
    }
}

// The whole selection of a small bank (at most SMALL_KEYS x 1024 templates, 32
// sub-bands) by one workgroup, the keys in registers: radix passes and counts
// in LDS, then the compaction.  One launch of 18 us in place of six with little
// work each (10800 templates, one sub-band: 120 us with the passes' launches,
// fills and scans).  Above these limits the keys leave the registers.
constexpr int SMALL_KEYS = 16, SMALL_SEG = 32;

__global__ __launch_bounds__(1024) void select_small_kernel(const float *stats, const int32_t *seg_of, Rows rw, SelectBufs b,
                                                            int n_seg, int k, double two_e, uint32_t *err)
{
    extern __shared__ uint32_t hsh[];  // [n_seg][256]
    __shared__ uint32_t state[SMALL_SEG * ST], cnt[SMALL_SEG], off[SMALL_SEG + 1], fill[SMALL_SEG];
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t key[SMALL_KEYS];
    int sg[SMALL_KEYS];
#pragma unroll
    for (int i = 0; i < SMALL_KEYS; ++i) {
        const int t = tid + 1024 * i;
        sg[i] = -1;
        key[i] = 0;
        if (t < rw.n_total) {
            sg[i] = seg_of[rw.grid ? t % (int)rw.row_len : t];
            key[i] = __float_as_uint(stats[t]);
            if (key[i] > NAN_KEY) sg[i] = -1;
        }
    }
    if (tid < n_seg) {
        uint32_t *st = state + tid * ST;
        st[S_PREFIX] = st[S_MASK] = st[S_DONE] = st[S_THR] = 0;
        st[S_KREM] = (uint32_t)k;
        cnt[tid] = fill[tid] = 0;
    }
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int q = tid; q < n_seg * 256; q += 1024) hsh[q] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SMALL_KEYS; ++i) {
            int idx = -1;
            if (sg[i] >= 0) {
                const uint32_t *st = state + sg[i] * ST;
                if (!st[S_DONE] && (key[i] & st[S_MASK]) == st[S_PREFIX]) idx = sg[i] * 256 + (int)((key[i] >> shift) & 255u);
            }
            const uint64_t valid = __builtin_amdgcn_ballot_w64(idx >= 0);
            if (valid == 0) continue;
            const int first = __builtin_ctzll(valid);
            const int lead = __builtin_amdgcn_readlane(idx, first);
            if (__builtin_amdgcn_ballot_w64(idx == lead) == valid) {
                if (lane == first) atomicAdd(&hsh[lead], (uint32_t)__builtin_popcountll(valid));
            } else if (idx >= 0) {
                atomicAdd(&hsh[idx], 1u);
            }
        }
        __syncthreads();
        for (int q = tid >> 6; q < n_seg; q += 16) choose_digit([&](int d) { return hsh[q * 256 + d]; }, state + q * ST, shift, two_e);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < SMALL_KEYS; ++i)
        if (sg[i] >= 0 && key[i] >= state[sg[i] * ST + S_THR]) atomicAdd(&cnt[sg[i]], 1u);
    __syncthreads();
    if (tid == 0) {
        uint32_t acc = 0;
        off[0] = b.off[0] = 0;
        for (int q = 0; q < n_seg; ++q) {
            acc += cnt[q];
            off[q + 1] = b.off[q + 1] = acc;
            b.cnt[q] = cnt[q];
            b.n_out[q] = (int32_t)min(cnt[q], (uint32_t)k);
        }
        if ((int64_t)acc > b.cap) atomicOr(err, ERR_CAND_OVERFLOW);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SMALL_KEYS; ++i)
        if (sg[i] >= 0 && key[i] >= state[sg[i] * ST + S_THR]) {
            const int64_t pos = (int64_t)off[sg[i]] + atomicAdd(&fill[sg[i]], 1u);
            if (pos < b.cap) b.cand[pos] = tid + 1024 * i;
        }
}

// The evaluation's results into mapped host memory, as part of its sequence:
// reading a toplist then takes one wait instead of four copies of 10 to 35 us.
__global__ __launch_bounds__(256) void deliver_kernel(const uint32_t *err, int n_seg, int k, SelectBufs b, DeliverHead *head,
                                                      int32_t *n_out, uint64_t *out)
{
    constexpr int W = sizeof(ft_candidate) / 8;
    static_assert(sizeof(ft_candidate) % 8 == 0, "entries are copied in words of 8 bytes");
    const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    if (i0 == 0) head->flags = *err;
    for (int64_t sg = i0; sg < n_seg; sg += step) n_out[sg] = b.n_out[sg];
    const uint64_t *src = (const uint64_t *)b.out;
    const int64_t row = (int64_t)k * W;
    for (int64_t w = i0; w < n_seg * row; w += step)
        if (w % row / W < b.n_out[w / row]) out[w] = src[w];
}

// ---------------------------------------------------------------------------
// Batches: one workgroup per run does the whole exact selection of that run
// (runs hold at most a few 1e5 templates): radix select in LDS, candidate
// compaction, FP64 re-summation and ranking.  A wave chooses a digit (a lane
// alone took 55 us over a run's four).  A run's five passes over its keys wait
// on memory and on the histogram's cells: sixteen keys are read ahead and equal
// digits of a wave added together (64 runs of up to 10^5 templates: 249 us with
// eight and an atomic a key, 181 us).
//
// The re-summation is a chain of 256 terms at a time: 1.7 us for a wave that
// forms and adds them, 2.7 us per 768 terms and two more such steps for a group
// of four (three form, one adds).  So a group each takes a run's candidates only
// where there are as few and the run is long (64 runs of up to 10^4 SFTs, one
// candidate: 67 us, a wave each 94 us; up to 1000 SFTs: 195 and 82; 10^4 SFTs
// and 512 candidates: 10.3 and 8.8 ms).
// ---------------------------------------------------------------------------
constexpr int SB_GROUP_WAVES = 4, SB_LONG = 1536;
constexpr int SB_AHEAD = 16;

template <int SB_GROUPS>
__global__ __launch_bounds__(256 * SB_GROUPS) void select_batch_kernel(const EvalRun *runs, int k, int cap,
                                                                int64_t *cand_all, double *s64_all,
                                                                ft_candidate *out, int32_t *n_out,
                                                                double *max_z, uint32_t *err)
{
    constexpr int SB_THREADS = 256 * SB_GROUPS;
    __shared__ uint32_t hist[256], st[ST], n_cand;
    __shared__ SeqBuf<SB_GROUP_WAVES, false> seq[SB_GROUPS];
    const int r = blockIdx.x;
    const EvalRun R = runs[r];
    const int64_t n_t = (int64_t)R.n_f0 * R.n_f1 * R.n_sky;
    const int tid = threadIdx.x;
    const double N = (double)R.n_sft;
    const double two_e = 2.0 * (40.0 * 0x1p-24 + 4.0 * N * 0x1p-53);
    int64_t *cand = cand_all + (int64_t)r * cap;
    double *s64 = s64_all + (int64_t)r * cap;
    if (tid == 0) {
        st[S_PREFIX] = st[S_MASK] = st[S_DONE] = st[S_THR] = 0;
        st[S_KREM] = (uint32_t)k;
        n_cand = 0;
    }
    // f(t, key) for every template's statistic that is a number
    auto keys = [&](auto f) {
        for (int64_t t0 = tid; t0 < n_t; t0 += SB_AHEAD * SB_THREADS) {
            uint32_t key[SB_AHEAD];
#pragma unroll
            for (int i = 0; i < SB_AHEAD; ++i)
                key[i] = t0 + i * SB_THREADS < n_t ? __float_as_uint(R.stats[t0 + i * SB_THREADS]) : ~0u;
#pragma unroll
            for (int i = 0; i < SB_AHEAD; ++i)
                if (key[i] <= NAN_KEY) f(t0 + i * SB_THREADS, key[i]);
        }
    };
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        if (!st[S_DONE]) {
            const uint32_t mask = st[S_MASK], prefix = st[S_PREFIX];
            keys([&](int64_t, uint32_t key) {
                if ((key & mask) != prefix) return;
                // a run's keys share their leading digit, and atomics to one
                // cell are performed one lane at a time: the lanes that agree
                // with the first add their number together
                const uint32_t d = (key >> shift) & 255u, lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
                const uint64_t same = __builtin_amdgcn_ballot_w64(d == lead);
                if (d != lead) atomicAdd(&hist[d], 1u);
                else if ((tid & 63) == __builtin_ctzll(same)) atomicAdd(&hist[d], (uint32_t)__builtin_popcountll(same));
            });
        }
        __syncthreads();
        if (tid < 64) choose_digit([&](int d) { return hist[d]; }, st, shift, two_e);
        __syncthreads();
    }
    const uint32_t thr = st[S_THR];
    keys([&](int64_t t, uint32_t key) {
        if (key < thr) return;
        const uint32_t pos = atomicAdd(&n_cand, 1u);
        if (pos < (uint32_t)cap) cand[pos] = t;
    });
    __syncthreads();
    int nc = (int)n_cand;
    if (nc > cap) {
        if (tid == 0) atomicOr(err, ERR_CAND_OVERFLOW);
        nc = cap;
    }
    // FP64 re-summation in SFT order with canonical bins
    uint32_t bad = 0;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), group = wave / SB_GROUP_WAVES;
    if (nc > 0 && nc <= SB_GROUPS && R.n_sft > SB_LONG) {
        const TemplateParams tp = params_of(R, true, cand[min(group, nc - 1)]);
        double acc, d0, d1;
        seq_sums<SB_GROUP_WAVES, false>(
            [&](int k_sft, float (&pw)[4], double (&w)[4]) { rescore_terms(R, tp, k_sft, false, 0.0, bad, pw, w); },
            R.n_sft, seq[group], wave % SB_GROUP_WAVES, group < nc, acc, d0, d1);
        if (group < nc && tid % (64 * SB_GROUP_WAVES) == 0) s64[group] = acc;
    } else {
        double *buf = seq[group].val[0] + 64 * RS_UNROLL * (wave % SB_GROUP_WAVES);
        static_assert(64 * RS_UNROLL * SB_GROUP_WAVES <= 2 * SeqBuf<SB_GROUP_WAVES, false>::CH, "a slice a wave");
        for (int p = wave; p < nc; p += SB_GROUP_WAVES * SB_GROUPS) {
            const double acc = rescore_wave(R, true, cand[p], tid & 63, bad, buf);
            if ((tid & 63) == 0) s64[p] = acc;
        }
    }
    if (bad) atomicOr(err, bad);
    __syncthreads();
    const double mu = 2.0 * N, sigma = 2.0 * sqrt(N);
    for (int p = tid; p < nc; p += SB_THREADS) {
        const double sp = s64[p];
        const int64_t tp = cand[p];
        int rank = 0;
        for (int q = 0; q < nc && rank < k; ++q) {
            const double sq = s64[q];
            rank += (sq > sp) || (sq == sp && cand[q] < tp);
        }
        if (rank < k) {
            const TemplateParams par = params_of(R, true, tp);
            ft_candidate c;
            c.index = tp;
            c.sub = 0;
            c.s32 = R.stats[tp];
            c.f0 = par.f0;
            c.f1 = par.f1;
            c.n[0] = par.nx;
            c.n[1] = par.ny;
            c.n[2] = par.nz;
            c.s64 = sp;
            c.z = (sp - mu) / sigma;
            out[(int64_t)r * k + rank] = c;
            if (rank == 0) max_z[r] = c.z;
        }
    }
    if (tid == 0) n_out[r] = min(nc, k);
}

__global__ void labels_kernel(const double *max_z, int n_runs, double tau, uint8_t *labels)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n_runs) labels[r] = max_z[r] > tau ? 1 : 0;
}

Rows rows_of(const EvalRun &r, bool grid)
{
    Rows rw;
    rw.grid = grid;
    if (grid) {
        rw.row_len = r.n_f0;
        rw.n_rows = (int64_t)r.n_sky * r.n_f1;
        rw.n_total = rw.n_rows * rw.row_len;
    } else {
        // rows of 256 templates and up, so that a bank of 1e5 has some 400
        rw.row_len = 256 * std::min<int64_t>(std::max<int64_t>(r.n_list / (256 * 1024), 1), 16);
        rw.n_total = r.n_list;
        rw.n_rows = (r.n_list + rw.row_len - 1) / rw.row_len;
    }
    return rw;
}

// Workgroups of a pass: each adds its histogram to the sub-bands' with atomics
// that are performed one by one, so the fewer the better while the keys fit the
// caches (grid of 1.6e6: selection 92 us with 512, 118 us with 2048; list of
// 2e6: 173 us and 151 us); larger banks are read from memory and need them all
// (4e7: 826 us and 421 us).
unsigned blocks_for(const Rows &rw)
{
    const int64_t most = rw.n_total <= (1 << 21) ? 512 : 2048;
    return (unsigned)std::min(std::max<int64_t>(rw.n_rows, 1), most);
}

}  // namespace

hipError_t launch_select_batch(const EvalRun *runs, int n_runs, int64_t max_t, int k, int cap_per_run,
                               int64_t *cand, double *cand_s64, ft_candidate *out,
                               int32_t *n_out, double *max_z, uint32_t *err, hipStream_t s)
{
    if (n_runs <= 0) return hipSuccess;
    // few candidates and keys a run, and runs for every CU: a group each, so that
    // four and more runs share a CU.  Toplists of one, with four groups and one:
    // 1024 runs of 880 templates and 10^4 SFTs 435 and 304 us; short runs, 300 of
    // 1000 templates 38 and 26, of 4000 39 and 54, of 2 10^5 392 and 841; 1024 of
    // 4000 102 and 79, of 16,000 145 and 177
    const bool small = k <= 2 && n_runs > 256 && max_t <= 8 * (int64_t)n_runs;
    auto *kern = small ? select_batch_kernel<1> : select_batch_kernel<4>;
    const int threads = small ? 256 : 1024;
    hipLaunchKernelGGL(kern, dim3((unsigned)n_runs), dim3(threads), 0, s, runs, k, cap_per_run, cand, cand_s64, out, n_out,
                       max_z, err);
    return hipGetLastError();
}

hipError_t launch_labels(const double *max_z, int n_runs, double tau, uint8_t *labels,
                         hipStream_t s)
{
    if (n_runs <= 0) return hipSuccess;
    hipLaunchKernelGGL(labels_kernel, dim3((unsigned)((n_runs + 255) / 256)), dim3(256), 0, s,
                       max_z, n_runs, tau, labels);
    return hipGetLastError();
}

static bool small_select(const Rows &rw, int n_seg) { return rw.n_total <= 1024 * SMALL_KEYS && n_seg <= SMALL_SEG; }

hipError_t launch_select_prep(const double *f0, int64_t n, const double *edges, int n_seg, int32_t *seg, int k,
                              const SelectBufs &b, uint32_t *err, hipStream_t s)
{
    const unsigned g = (unsigned)std::min<int64_t>((std::max<int64_t>(n, (int64_t)n_seg * 256) + 255) / 256, 4096);
    hipLaunchKernelGGL(select_prep_kernel, dim3(g), dim3(256), 0, s, f0, n, edges, n_seg, seg, k, b, err);
    return hipGetLastError();
}

hipError_t launch_select(const EvalRun &r, bool grid, int n_seg, int k, double rel_err,
                         const SelectBufs &b, hipStream_t s)
{
    const Rows rw = rows_of(r, grid);
    const double two_e = 2.0 * rel_err;
    if (small_select(rw, n_seg)) {
        hipLaunchKernelGGL(select_small_kernel, dim3(1), dim3(1024), (size_t)n_seg * 256 * sizeof(uint32_t), s, r.stats,
                           b.seg_of_f0, rw, b, n_seg, k, two_e, r.err);
        return hipGetLastError();
    }
    const bool lds_hist = n_seg * 256 <= 8192;
    const unsigned nb = blocks_for(rw);
    // grid rows of at most 2048 templates: column-owning kernels
    const int cols = !grid || !lds_hist ? 0 : rw.row_len <= 1024 ? 4 : rw.row_len <= 2048 ? 8 : 0;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        uint32_t *hist = b.hist + (int64_t)pass * n_seg * 256, *ticket = b.ticket + pass * SEL_TICKET;
        const size_t hl = (size_t)n_seg * 256 * sizeof(uint32_t);
        if (cols == 4)
            hipLaunchKernelGGL(hist_grid_kernel<4>, dim3(nb), dim3(256), hl, s, r.stats, b.seg_of_f0, rw, b.state,
                               hist, n_seg, shift, two_e, ticket);
        else if (cols == 8)
            hipLaunchKernelGGL(hist_grid_kernel<8>, dim3(nb), dim3(256), hl, s, r.stats, b.seg_of_f0, rw, b.state,
                               hist, n_seg, shift, two_e, ticket);
        else if (lds_hist)
            hipLaunchKernelGGL(hist_kernel<true>, dim3(nb), dim3(256), hl, s, r.stats, b.seg_of_f0, rw, b.state, hist,
                               n_seg, shift, two_e, ticket);
        else {
            hipLaunchKernelGGL(hist_kernel<false>, dim3(nb), dim3(256), 0, s, r.stats, b.seg_of_f0, rw, b.state, hist,
                               n_seg, shift, two_e, ticket);
            hipLaunchKernelGGL(digits_kernel, dim3((unsigned)((n_seg + 3) / 4)), dim3(256), 0, s, b.state, hist, n_seg,
                               shift, two_e);
        }
    }
    const size_t cl = (size_t)n_seg * sizeof(uint32_t);
    if (cols == 4)
        hipLaunchKernelGGL(count_grid_kernel<4>, dim3(nb), dim3(256), cl, s, r.stats, b.seg_of_f0, rw, b.state, b, n_seg,
                           k, r.err);
    else if (cols == 8)
        hipLaunchKernelGGL(count_grid_kernel<8>, dim3(nb), dim3(256), cl, s, r.stats, b.seg_of_f0, rw, b.state, b, n_seg,
                           k, r.err);
    else
        hipLaunchKernelGGL(count_kernel, dim3(nb), dim3(256), cl, s, r.stats, b.seg_of_f0, rw, b.state, b, n_seg, k,
                           r.err);
    if (cols == 4)
        hipLaunchKernelGGL(scatter_grid_kernel<4>, dim3(nb), dim3(256), 0, s, r.stats, b.seg_of_f0, rw, b.state,
                           b.off, b.fill, b.cand, b.cap);
    else if (cols == 8)
        hipLaunchKernelGGL(scatter_grid_kernel<8>, dim3(nb), dim3(256), 0, s, r.stats, b.seg_of_f0, rw, b.state,
                           b.off, b.fill, b.cand, b.cap);
    else
        hipLaunchKernelGGL(scatter_kernel, dim3(nb), dim3(256), 0, s, r.stats, b.seg_of_f0, rw,
                           b.state, b.off, b.fill, b.cand, b.cap);
    return hipGetLastError();
}

// Re-summation of the candidates, about `expect` of them: a workgroup each up to
// 1024, a wave each beyond.  Over 10^4 SFTs with a workgroup each and a wave each:
// 250 candidates 33 and 67 us, 1000 65 and 62 (binary banks 70 and 81), 3000 181
// and 163, 10^4 730 and 547; over 30 SFTs, 4000: 22 and 10.
static void launch_rescore(const EvalRun &r, bool grid, const int64_t *cand, const uint32_t *off, int n_seg, int64_t cap,
                           int64_t expect, double *s64, double *mom, hipStream_t s)
{
    if (mom)
        hipLaunchKernelGGL(rescore_kernel<true>, dim3(2048), dim3(64 * RS_WAVES), 0, s, r, grid, cand, off, n_seg, cap,
                           s64, mom);
    else if (expect <= 1024)
        hipLaunchKernelGGL(rescore_kernel<false>, dim3(2048), dim3(64 * RS_WAVES), 0, s, r, grid, cand, off, n_seg, cap,
                           s64, mom);
    else
        hipLaunchKernelGGL(rescore_many_kernel, dim3(2048), dim3(256), 0, s, r, grid, cand, off, n_seg, cap, s64);
}

hipError_t launch_deliver(const uint32_t *err, int n_seg, int k, const SelectBufs &b, char *host, hipStream_t s)
{
    const int64_t words = (int64_t)n_seg * k * (int64_t)(sizeof(ft_candidate) / 8);
    const unsigned g = (unsigned)std::min<int64_t>((words + 255) / 256, 256);
    hipLaunchKernelGGL(deliver_kernel, dim3(g), dim3(256), 0, s, err, n_seg, k, b, (DeliverHead *)host,
                       (int32_t *)(host + sizeof(DeliverHead)), (uint64_t *)(host + deliver_entries_at(n_seg)));
    return hipGetLastError();
}

hipError_t launch_rescore_rank(const EvalRun &r, bool grid, int n_seg, int k,
                               const SelectBufs &b, hipStream_t s)
{
    double *mom = !grid && r.arms ? b.cand_mom : nullptr;  // binary banks with sky weights
    launch_rescore(r, grid, b.cand, b.off, n_seg, b.cap, (int64_t)n_seg * k, b.cand_s64, mom, s);
    hipLaunchKernelGGL(rank_kernel, dim3(1024), dim3(256), 0, s, r, grid, b.cand, b.cand_s64,
                       b.off, n_seg, b.cap, k, b.mu_sigma, mom, b.out);
    return hipGetLastError();
}

// --- loudest template per hyperbox ------------------------------------------
__global__ void box_init_kernel(int64_t n_boxes, uint32_t *max32, int32_t *count, unsigned long long *max64,
                                unsigned long long *idx, uint32_t *n_cand)
{
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n_boxes;
         b += (int64_t)gridDim.x * blockDim.x) {
        max32[b] = 0u;
        count[b] = 0;
        max64[b] = 0ull;
        idx[b] = ~0ull;
    }
    if (blockIdx.x == 0 && threadIdx.x < 2) n_cand[threadIdx.x] = 0u;
}

// Statistics are >= 0, so their bit patterns order like their values.
__global__ void box_max_kernel(const float *stats, const int32_t *box, int64_t n, uint32_t *max32, int32_t *count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = box[i];
        atomicMax(max32 + b, __float_as_uint(stats[i]));
        atomicAdd(count + b, 1);
    }
}

// Candidates: S32 >= max32 (1 - 2 rel_err).  The template with the largest
// S64 of a box has S32 >= S64 (1 - rel) and the box's FP32 maximum is at most
// S64max (1 + rel), so it is always kept.
__global__ void box_cand_kernel(const float *stats, const int32_t *box, int64_t n, const uint32_t *max32, double keep,
                                int64_t *cand, uint32_t *n_cand, int64_t cap, uint32_t *err)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double thr = (double)__uint_as_float(max32[box[i]]) * keep;
        if ((double)stats[i] >= thr) {
            const uint32_t pos = atomicAdd(n_cand + 1, 1u);
            if (pos < cap) cand[pos] = i;
            else atomicOr(err, ERR_CAND_OVERFLOW);
        }
    }
}

__global__ void box_pick_kernel(const int64_t *cand, const double *s64, const uint32_t *n_cand, int64_t cap,
                                const int32_t *box, unsigned long long *max64)
{
    const int64_t total = min((int64_t)n_cand[1], cap);
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += (int64_t)gridDim.x * blockDim.x)
        atomicMax(max64 + box[cand[p]], (unsigned long long)__double_as_longlong(s64[p]));
}

__global__ void box_index_kernel(const int64_t *cand, const double *s64, const uint32_t *n_cand, int64_t cap,
                                 const int32_t *box, const unsigned long long *max64, unsigned long long *idx)
{
    const int64_t total = min((int64_t)n_cand[1], cap);
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = box[cand[p]];
        if ((unsigned long long)__double_as_longlong(s64[p]) == max64[b]) atomicMin(idx + b, (unsigned long long)cand[p]);
    }
}

__global__ void box_out_kernel(int64_t n_boxes, const int32_t *count, const unsigned long long *max64,
                               const unsigned long long *idx, const float *stats, const double *mu_sigma,
                               ft_box_result *out)
{
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n_boxes;
         b += (int64_t)gridDim.x * blockDim.x) {
        ft_box_result r;
        r.count = count[b];
        if (r.count > 0) {
            r.index = (int64_t)idx[b];
            r.s32 = stats[r.index];
            r.s64 = __longlong_as_double((long long)max64[b]);
            r.z = (r.s64 - mu_sigma[0]) / mu_sigma[1];
        } else {
            r.index = -1;
            r.s32 = 0.f;
            r.s64 = 0.0;
            r.z = 0.0;
        }
        out[b] = r;
    }
}

hipError_t launch_box_max(const EvalRun &r, int64_t n, int64_t n_boxes, const BoxBufs &b, double rel_err,
                          hipStream_t s)
{
    const unsigned gb = (unsigned)std::min<int64_t>((n_boxes + 255) / 256, 8192);
    const unsigned gn = (unsigned)std::min<int64_t>((n + 255) / 256, 16384);
    hipLaunchKernelGGL(box_init_kernel, dim3(gb > 0 ? gb : 1), dim3(256), 0, s, n_boxes, b.max32, b.count, b.max64,
                       b.idx, b.n_cand);
    if (n <= 0) return hipGetLastError();
    hipLaunchKernelGGL(box_max_kernel, dim3(gn), dim3(256), 0, s, r.stats, b.box, n, b.max32, b.count);
    hipLaunchKernelGGL(box_cand_kernel, dim3(gn), dim3(256), 0, s, r.stats, b.box, n, b.max32, 1.0 - 2.0 * rel_err,
                       b.cand, b.n_cand, b.cap, r.err);
    return hipGetLastError();
}

hipError_t launch_box_pick(const EvalRun &r, int64_t n_boxes, const BoxBufs &b, const double *mu_sigma,
                           ft_box_result *out, hipStream_t s)
{
    const unsigned gb = (unsigned)std::min<int64_t>((n_boxes + 255) / 256, 8192);
    launch_rescore(r, false, b.cand, b.n_cand, 1, b.cap, n_boxes, b.cand_s64, nullptr, s);
    hipLaunchKernelGGL(box_pick_kernel, dim3(1024), dim3(256), 0, s, b.cand, b.cand_s64, b.n_cand, b.cap, b.box,
                       b.max64);
    hipLaunchKernelGGL(box_index_kernel, dim3(1024), dim3(256), 0, s, b.cand, b.cand_s64, b.n_cand, b.cap, b.box,
                       b.max64, b.idx);
    hipLaunchKernelGGL(box_out_kernel, dim3(gb > 0 ? gb : 1), dim3(256), 0, s, n_boxes, b.count, b.max64, b.idx,
                       r.stats, mu_sigma, out);
    return hipGetLastError();
}

hipError_t launch_rescore_entries(const EvalRun &r, bool grid, const ft_candidate *top, const int32_t *n_out,
                                  double *out, hipStream_t s)
{
    hipLaunchKernelGGL(rescore_entries_kernel, dim3(256), dim3(64 * RS_WAVES), 0, s, r, grid, top, n_out, out);
    return hipGetLastError();
}

}  // namespace ft
