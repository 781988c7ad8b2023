// fishnet.hip -- gfx950 kernels of fishnet casting (Section 2.5, Algorithm 7).
//
// Up to PS candidate points run fixed-step PDHG together on the scaled LP.
// The points are interleaved (entry r of point q at [r * PS + q]), and a row
// of K~ (or K~^T) is handled by a group of j lanes, lane q for point q, where
// j is the number of live points (a power of two <= 64).  Every lane of the
// group loads the same matrix entry (one transaction for the group) and
// gathers point q's entry of the column, so a gather moves j contiguous
// values: the multi-point sweep reads the matrix once for all points.  A sweep
// of few points is bound by its chains of dependent loads, not by traffic (at
// 1.5M entries the two sweeps of an iteration took 23 + 41 us with one lane per
// point and row), so 2^ls lanes share a point's row, each reading quads of
// entries two at a time, and rows of more than FISH_LONG entries take a whole
// workgroup: 25 + 24 us at 32 points, 11 + 16 us at 4.  Rows longer than
// FISH_CHUNK entries are cut into chunks (their partial sums are added by a
// combine pass in chunk order), and the tasks run longest first.  The sums'
// order depends on the row's length, the number of rows and of live points only.
//
// One round: k primal/dual steps on the live points, the duality gap of each
// point (grid-stride partials, reduced in a fixed order), a one-workgroup
// ranking that keeps the better half (ties by index) and, in odd rounds that
// start with more than two points, builds the repopulation weights, then a
// gather pass that writes the next round's points: the kept ones (best first)
// followed by the new convex combinations.
#include <hip/hip_runtime.h>
#include <math.h>

#include "../../include/pdhg.h"
#include "kernels.h"
#include "sweep.h"

namespace pdhg {

// Four consecutive entries, loaded at any alignment of one entry.
typedef int32_t Cols4 __attribute__((ext_vector_type(4), aligned(4)));
template <typename V>
struct Vals4;
template <>
struct Vals4<float> {
    typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct Vals4<double> {
    typedef double type __attribute__((ext_vector_type(4), aligned(8)));
};

// This lane's share of a row's sum over entries [b, e) for its point: quads
// s, s + S, ... of the row (the last one may hold fewer than four entries), two
// of them in flight.  G points at the lane's point in entry 0.
template <typename MV, typename GV>
__device__ __forceinline__ double fish_dot(const OpDev &op, const MV *__restrict__ va, int64_t b, int64_t e,
                                           const GV *__restrict__ G, int PS, int s, int S)
{
    using V4 = typename Vals4<MV>::type;
    const int32_t *__restrict__ ci = op.ci;
    const int st = 4 * S;
    double acc = 0.0;
    int64_t p = b + 4 * s;
    for (; p + st + 4 <= e; p += 2 * st) {
        const Cols4 c0 = *(const Cols4 *)(ci + p), c1 = *(const Cols4 *)(ci + p + st);
        const V4 v0 = *(const V4 *)(va + p), v1 = *(const V4 *)(va + p + st);
        GV g[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) g[k] = G[(int64_t)c0[k] * PS];
#pragma unroll
        for (int k = 0; k < 4; ++k) g[4 + k] = G[(int64_t)c1[k] * PS];
#pragma unroll
        for (int k = 0; k < 4; ++k) acc += (double)v0[k] * (double)g[k];
#pragma unroll
        for (int k = 0; k < 4; ++k) acc += (double)v1[k] * (double)g[4 + k];
    }
    if (p + 4 <= e) {
        const Cols4 c0 = *(const Cols4 *)(ci + p);
        const V4 v0 = *(const V4 *)(va + p);
        GV g[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) g[k] = G[(int64_t)c0[k] * PS];
#pragma unroll
        for (int k = 0; k < 4; ++k) acc += (double)v0[k] * (double)g[k];
        p += st;
    }
    for (; p < e; ++p) acc += (double)va[p] * (double)G[(int64_t)ci[p] * PS];
    return acc;
}

// Sum over the lanes of one point in a wavefront: bits [lj, top) of the lane.
__device__ __forceinline__ double fish_sum(double v, int lj, int top)
{
    for (int off = 1 << lj; off < (1 << top); off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// x+ = clip(x - tau (c~ - g), l~, u~), xbar = 2 x+ - x
template <typename T>
__device__ __forceinline__ void fish_primal_epi(const Dev &d, const FishDev &f, int64_t row, int q, double g,
                                                double tau)
{
    T *X = (T *)f.X;
    const int64_t at = row * f.PS + q;
    const double xo = (double)X[at];
    const double v = xo - tau * ((double)((const T *)d.c)[row] - g);
    const double lo = (double)((const T *)d.l)[row], hi = (double)((const T *)d.u)[row];
    const T xn = (T)(v < lo ? lo : (v > hi ? hi : v));
    X[at] = xn;
    ((T *)f.XB)[at] = (T)(2.0 * (double)xn - xo);
}

// INIT = 0: y+ = proj_Y(y + sigma (q~ - r)); INIT = 1: y = r
template <typename T, int INIT>
__device__ __forceinline__ void fish_dual_epi(const Dev &d, const FishDev &f, int64_t row, int q, double r,
                                              double sigma, int64_t m1)
{
    T *Y = (T *)f.Y;
    const int64_t at = row * f.PS + q;
    if (INIT) {
        Y[at] = (T)r;
        return;
    }
    const double w = (double)Y[at] + sigma * ((double)((const T *)d.q)[row] - r);
    Y[at] = (T)((row < m1 && w < 0.0) ? 0.0 : w);
}

// The task of this lane and its sum: a task of the first nlong takes a whole
// workgroup (WG / j lanes per point), every other one a group of 2^(lj + ls)
// lanes of a wavefront.  True in the lanes that hold the sum of a task.
template <typename T>
__device__ __forceinline__ bool fish_task(const OpDev &op, const int4 *task, int64_t ntask, int64_t nlong,
                                          const T *__restrict__ G, int PS, int lj, int ls, double *lds, int4 &t,
                                          double &acc)
{
    const int tid = threadIdx.x, q = tid & ((1 << lj) - 1), s = tid >> lj;
    if (blockIdx.x < nlong) {
        t = task[blockIdx.x];
        acc = fish_sum(fish_dot(op, op_vals<T>(op), t.y, t.z, G + q, PS, s, WG >> lj), lj, 6);
        const int wave = tid >> 6, lane = tid & 63;
        if (lane >> lj == 0) lds[wave * 64 + lane] = acc;
        __syncthreads();
        if (s) return false;
        acc = (lds[q] + lds[64 + q]) + (lds[128 + q] + lds[192 + q]);
        return true;
    }
    const int lg = lj + ls;
    const int64_t g = nlong + (blockIdx.x - nlong) * (WG >> lg) + (tid >> lg);
    if (g >= ntask) return false;
    t = task[g];
    const int sl = s & ((1 << ls) - 1);
    acc = fish_sum(fish_dot(op, op_vals<T>(op), t.y, t.z, G + q, PS, sl, 1 << ls), lj, lg);
    return sl == 0;
}

// A task that covers its whole row applies the update; a chunk of a split
// row stores its partial sum for the combine pass.
template <typename T>
__global__ __launch_bounds__(WG) void k_fish_primal(Dev d, FishDev f, int lj, int ls, double tau)
{
    __shared__ double lds[256];
    const int q = threadIdx.x & ((1 << lj) - 1);
    int4 t;
    double acc;
    if (!fish_task(d.Kt, f.taskT, f.ntaskT, f.nlongT, (const T *)f.Y, f.PS, lj, ls, lds, t, acc)) return;
    if (t.w < 0)
        fish_primal_epi<T>(d, f, t.x, q, acc, tau);
    else
        f.cpart[(int64_t)t.w * f.PS + q] = acc;
}

template <typename T, int INIT>
__global__ __launch_bounds__(WG) void k_fish_dual(Dev d, FishDev f, int lj, int ls, double sigma, int64_t m1)
{
    __shared__ double lds[256];
    const int q = threadIdx.x & ((1 << lj) - 1);
    int4 t;
    double acc;
    if (!fish_task(d.K, f.taskK, f.ntaskK, f.nlongK, (const T *)(INIT ? f.X : f.XB), f.PS, lj, ls, lds, t, acc))
        return;
    if (t.w < 0)
        fish_dual_epi<T, INIT>(d, f, t.x, q, acc, sigma, m1);
    else
        f.cpart[(int64_t)t.w * f.PS + q] = acc;
}

// Combine passes: the chunk partials of each split row, in chunk order.
template <typename T>
__global__ __launch_bounds__(WG) void k_fish_combine_primal(Dev d, FishDev f, int lj, double tau)
{
    const int tid = threadIdx.x, q = tid & ((1 << lj) - 1);
    const int64_t g = (int64_t)blockIdx.x * (WG >> lj) + (tid >> lj);
    if (g >= f.nsplitT) return;
    const int4 sp = f.splitT[g];
    double acc = 0.0;
    for (int c = 0; c < sp.z; ++c) acc += f.cpart[(int64_t)(sp.y + c) * f.PS + q];
    fish_primal_epi<T>(d, f, sp.x, q, acc, tau);
}

template <typename T, int INIT>
__global__ __launch_bounds__(WG) void k_fish_combine_dual(Dev d, FishDev f, int lj, double sigma, int64_t m1)
{
    const int tid = threadIdx.x, q = tid & ((1 << lj) - 1);
    const int64_t g = (int64_t)blockIdx.x * (WG >> lj) + (tid >> lj);
    if (g >= f.nsplitK) return;
    const int4 sp = f.splitK[g];
    double acc = 0.0;
    for (int c = 0; c < sp.z; ++c) acc += f.cpart[(int64_t)(sp.y + c) * f.PS + q];
    fish_dual_epi<T, INIT>(d, f, sp.x, q, acc, sigma, m1);
}

// Per-workgroup partials of dobj - pobj for every live point (scaled data,
// FP64 matrix): K~^T rows add l~ lambda^+ + u~ lambda^- - c~ x with
// lambda = proj_Lambda(c~ - K~^T y); K rows add q~ y.  Row groups are
// visited grid-stride, so each workgroup's sum has a fixed order.
template <typename T>
__global__ __launch_bounds__(WG) void k_fish_gap(Dev d, FishDev f, int lj, int ls, int64_t gT, int64_t gK)
{
    __shared__ double lds[4 * 64];
    const int j = 1 << lj, S = 1 << ls;
    const int tid = threadIdx.x, q = tid & (j - 1), sl = (tid >> lj) & (S - 1), rl = tid >> (lj + ls);
    const int rpw = WG >> (lj + ls);
    const int PS = f.PS;
    const T *X = (const T *)f.X;
    const T *Y = (const T *)f.Y;
    double v = 0.0;
    for (int64_t it = blockIdx.x; it < gT + gK; it += gridDim.x) {
        if (it < gT) {
            const int64_t g = it * rpw + rl;
            if (g < d.Kt.nrows) {
                const int64_t row = f.rowT[g];
                const double a =
                    fish_sum(fish_dot(d.Kt, d.Kt.v64, d.Kt.rp[row], d.Kt.rp[row + 1], Y + q, PS, sl, S), lj, lj + ls);
                const double cj = d.c64[row], lo = d.l64[row], hi = d.u64[row];
                const bool lf = isfinite(lo), uf = isfinite(hi);
                const double dd = cj - a;
                // proj_Lambda: {0} free, R^- upper only, R^+ lower only, R boxed
                const double lam = (!lf && !uf) ? 0.0 : (!lf ? fmin(dd, 0.0) : (!uf ? fmax(dd, 0.0) : dd));
                const double t = lam > 0.0 ? lo * lam : (lam < 0.0 ? hi * lam : 0.0);
                if (sl == 0) v += t - cj * (double)X[row * PS + q];
            }
        } else {
            const int64_t g = (it - gT) * WG + tid;  // one row per lane and point
            const int64_t row = g >> lj;
            if (row < d.K.nrows) v += d.q64[row] * (double)Y[row * PS + q];
        }
    }
    // lanes of one point: across the rows of a wavefront, then the four wavefronts
    for (int off = 32; off >= j; off >>= 1) v += __shfl_xor(v, off);
    const int wave = tid >> 6, lane = tid & 63;
    if (lane < j) lds[wave * 64 + lane] = v;
    __syncthreads();
    if (tid < j) f.part[(size_t)blockIdx.x * PS + tid] = (lds[tid] + lds[64 + tid]) + (lds[128 + tid] + lds[192 + tid]);
}

// One workgroup: gaps of the live points, the kept half (stable order by
// gap, then index), the round's record, and in repopulating rounds the
// weights w_as = |g_as| / sum_s |g_as| (equal weights for an all-zero row).
__global__ __launch_bounds__(WG) void k_fish_rank(FishDev f, int lj, int nparts, int round, int repop, int half,
                                                  int64_t wpos)
{
    __shared__ double lds[WG];
    __shared__ double gap[64];
    __shared__ int idx[64];
    const int j = 1 << lj;
    const int tid = threadIdx.x, q = tid & (j - 1), sl = tid >> lj, nsl = WG >> lj;
    const int PS = f.PS;
    double v = 0.0;
    for (int b = sl; b < nparts; b += nsl) v += f.part[(size_t)b * PS + q];
    lds[tid] = v;
    __syncthreads();
    if (tid < j) {
        double t = 0.0;
        for (int s = 0; s < nsl; ++s) t += lds[s * j + tid];
        gap[tid] = fabs(t);
        idx[tid] = tid;
    }
    __syncthreads();
    if (tid == 0) {
        for (int a = 1; a < j; ++a) {
            const int t = idx[a];
            int b = a - 1;
            while (b >= 0 && (gap[idx[b]] > gap[t] || (gap[idx[b]] == gap[t] && idx[b] > t))) {
                idx[b + 1] = idx[b];
                --b;
            }
            idx[b + 1] = t;
        }
        if (round < f.nrec) {
            for (int r = 0; r < PS; ++r) {
                f.rec_gaps[(size_t)round * PS + r] = r < j ? gap[r] : 0.0;
                f.rec_keep[(size_t)round * PS + r] = r < half ? idx[r] : -1;
            }
        }
        for (int r = 0; r < half; ++r) f.keep[r] = idx[r];
    }
    if (repop && tid < half) {
        const double *w = f.wstage + wpos + (int64_t)tid * half;
        double tot = 0.0;
        for (int s = 0; s < half; ++s) tot += fabs(w[s]);
        for (int s = 0; s < half; ++s)
            f.wmat[tid * (PS / 2) + s] = tot > 0.0 ? fabs(w[s]) / tot : 1.0 / half;
    }
}

// Next round's points: column t < half is kept point keep[t]; column
// half + a is sum_s w_as * (kept point s), accumulated in FP64.
template <typename T>
__global__ void k_fish_gather(FishDev f, int lnext, int half, int64_t N, int64_t M)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t row = t >> lnext;
    const int col = (int)(t & ((1 << lnext) - 1));
    if (row >= N + M) return;
    const bool onX = row < N;
    const int64_t r = onX ? row : row - N;
    const int PS = f.PS;
    const T *src = (const T *)(onX ? f.X : f.Y) + r * PS;
    T *dst = (T *)(onX ? f.X2 : f.Y2) + r * PS;
    if (col < half) {
        dst[col] = src[f.keep[col]];
        return;
    }
    const double *w = f.wmat + (col - half) * (PS / 2);
    double v = 0.0;
    for (int s = 0; s < half; ++s) v += w[s] * (double)src[f.keep[s]];
    dst[col] = (T)v;
}

// X^0 = sc * G (G in the caller's column order, point-major)
template <typename T>
__global__ void k_fish_init(Dev d, FishDev f, int lp, double sc)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = t >> lp;
    const int q = (int)(t & ((1 << lp) - 1));
    if (r >= d.N) return;
    ((T *)f.X)[r * f.PS + q] = (T)(sc * f.gstage[(int64_t)q * d.N + d.col_orig[r]]);
}

// the last point to FP64 scratch vectors (the caller then installs it)
template <typename T>
__global__ void k_fish_out(Dev d, FishDev f)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < d.N) d.vecN64[t] = (double)((const T *)f.X)[t * f.PS];
    if (t < d.M) d.vecM64[t] = (double)((const T *)f.Y)[t * f.PS];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned fish_groups(int64_t rows, int lj)
{
    const int64_t rpw = WG >> lj;
    return (unsigned)((rows + rpw - 1) / rpw);
}

// log2 of the lanes per point of a short task: doubled (up to 8) until the
// launch has FISH_LANES lanes.  More lanes shorten a task's chain of loads and
// fill the chip; past that they only add shuffles and repeat the task's set-up.
// 32 points on 41k + 30k rows, ms for 512 iterations with 1 / 2 / 8 lanes
// throughout and with this rule: 18.2 / 17.8 / 22.5 / 17.7; 16 points on 8k + 6k
// rows: 8.8 / 6.3 / 5.2 / 5.1; 4 points on 100k + 72k rows: 5.8 / 4.6 / 6.5 / 4.7.
// A task of up to 8 entries is one step of a lane, which has two quads in flight,
// and a longer one has quads for len / 4 lanes: 8 points on 20,000 rows of 8 entries
// and 30,000 of 5, ms for 128 iterations with up to 8 lanes 4.00, with one 3.39.
static inline int fish_split(int64_t ntask, int len, int lj)
{
    int ls = 0;
    if (len <= 8) return ls;
    while (ls < 3 && lj + ls < 6 && (ntask << (lj + ls)) < FISH_LANES && (4 << ls) < len) ++ls;
    return ls;
}

static inline unsigned fish_blocks(int64_t ntask, int64_t nlong, int lg)
{
    return (unsigned)nlong + fish_groups(ntask - nlong, lg);
}

template <typename T>
void launch_fish_step(const Dev &d, const FishDev &f, int lj, double tau, double sigma, int64_t m1, hipStream_t s)
{
    const int lsT = fish_split(f.ntaskT, f.lenT, lj), lsK = fish_split(f.ntaskK, f.lenK, lj);
    const unsigned tT = fish_blocks(f.ntaskT, f.nlongT, lj + lsT), cT = fish_groups(f.nsplitT, lj);
    const unsigned tK = fish_blocks(f.ntaskK, f.nlongK, lj + lsK), cK = fish_groups(f.nsplitK, lj);
    if (tT) hipLaunchKernelGGL(k_fish_primal<T>, dim3(tT), dim3(WG), 0, s, d, f, lj, lsT, tau);
    if (cT) hipLaunchKernelGGL(k_fish_combine_primal<T>, dim3(cT), dim3(WG), 0, s, d, f, lj, tau);
    if (tK) hipLaunchKernelGGL((k_fish_dual<T, 0>), dim3(tK), dim3(WG), 0, s, d, f, lj, lsK, sigma, m1);
    if (cK) hipLaunchKernelGGL((k_fish_combine_dual<T, 0>), dim3(cK), dim3(WG), 0, s, d, f, lj, sigma, m1);
}

template <typename T>
void launch_fish_init(const Dev &d, const FishDev &f, int lp, double sc, hipStream_t s)
{
    const int64_t tot = d.N << lp;
    if (tot > 0) hipLaunchKernelGGL(k_fish_init<T>, dim3((unsigned)((tot + WG - 1) / WG)), dim3(WG), 0, s, d, f, lp, sc);
    const int ls = fish_split(f.ntaskK, f.lenK, lp);
    const unsigned tK = fish_blocks(f.ntaskK, f.nlongK, lp + ls), cK = fish_groups(f.nsplitK, lp);
    if (tK) hipLaunchKernelGGL((k_fish_dual<T, 1>), dim3(tK), dim3(WG), 0, s, d, f, lp, ls, 0.0, (int64_t)0);
    if (cK) hipLaunchKernelGGL((k_fish_combine_dual<T, 1>), dim3(cK), dim3(WG), 0, s, d, f, lp, 0.0, (int64_t)0);
}

template <typename T>
int launch_fish_gap_rank(const Dev &d, const FishDev &f, int lj, int round, int repop, int half, int64_t wpos,
                         hipStream_t s)
{
    const int ls = fish_split(f.ntaskT, f.lenT, lj);
    const int64_t gT = fish_groups(d.Kt.nrows, lj + ls), gK = fish_groups(d.K.nrows, lj);
    const int64_t items = gT + gK;
    const int grid = (int)(items < FISH_GRID ? (items > 0 ? items : 1) : FISH_GRID);
    hipLaunchKernelGGL(k_fish_gap<T>, dim3(grid), dim3(WG), 0, s, d, f, lj, ls, gT, gK);
    hipLaunchKernelGGL(k_fish_rank, dim3(1), dim3(WG), 0, s, f, lj, grid, round, repop, half, wpos);
    return grid;
}

template <typename T>
void launch_fish_gather(const Dev &d, const FishDev &f, int lnext, int half, hipStream_t s)
{
    const int64_t tot = (d.N + d.M) << lnext;
    if (tot > 0)
        hipLaunchKernelGGL(k_fish_gather<T>, dim3((unsigned)((tot + WG - 1) / WG)), dim3(WG), 0, s, f, lnext, half,
                           d.N, d.M);
}

template <typename T>
void launch_fish_out(const Dev &d, const FishDev &f, hipStream_t s)
{
    const int64_t n = d.N > d.M ? d.N : d.M;
    if (n > 0) hipLaunchKernelGGL(k_fish_out<T>, dim3((unsigned)((n + WG - 1) / WG)), dim3(WG), 0, s, d, f);
}

#define FISH_INST(T)                                                                                       \
    template void launch_fish_step<T>(const Dev &, const FishDev &, int, double, double, int64_t, hipStream_t); \
    template void launch_fish_init<T>(const Dev &, const FishDev &, int, double, hipStream_t);           \
    template int launch_fish_gap_rank<T>(const Dev &, const FishDev &, int, int, int, int, int64_t, hipStream_t); \
    template void launch_fish_gather<T>(const Dev &, const FishDev &, int, int, hipStream_t);            \
    template void launch_fish_out<T>(const Dev &, const FishDev &, hipStream_t);
FISH_INST(float)
FISH_INST(double)

}  // namespace pdhg
