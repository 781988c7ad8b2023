// small.hip -- fixed-step iterations of small LPs, many per launch.
//
// A sweep of a small LP is a launch and a chain of dependent loads (3-5 us)
// around a few hundred nanoseconds of work, and an iteration needs two of them.
// Here one 1024-lane workgroup per instance runs the iterations of a check
// period in one launch: the iterate, xbar, y and the averages stay in LDS and a
// workgroup barrier takes the place of the kernel boundary.
//
// One CU issues about one wavefront instruction per cycle, so what bounds it is
// the instruction count: the rows are laid out anew (small_rows_layout() in
// capi.cpp), sorted by length and taken 64 lanes at a time ("tasks") with one
// lane per row wherever rows are short, so that the update of a row runs in a
// full wavefront and few slots are padding; entry k of a task's 64 lanes is
// contiguous.  The layout, the columns (16 bit, relative to the instance) and
// the updates' operands are copied to LDS once per launch as far as they fit.
//
// A row's sum is formed as in tile.hip (fours of entries, dealt out to the row's
// lanes there; a lane here keeps 1, 2 or 4 of those lanes' partial sums and
// adds them in their order): the results are the same bit for bit, and a batch
// of small and larger LPs takes tile.hip for all of them.
//
// Measured, us per iteration (two launches / here): FP64 200 x 500 with 2.0k
// nonzeros 7.7 / 1.4; FP32 1003 x 2501 with 12.5k nonzeros 9.5 / 4.0.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "sweep.h"

namespace pdhg {
namespace {

// One operator's slots: in LDS or global memory.
template <typename T>
struct SmallSlots {
    const T *val;
    const uint16_t *col;
    const uint16_t *row;  // LDS: 64 row numbers per task
    // {first slot, entries per lane, lanes_log2 | sums_log2 << 8, rows}: constant
    // memory, so that a task's line comes through the scalar cache
    const __attribute__((address_space(4))) int32_t *task;
    int ntask;
};

// the products of U (<= 4) consecutive entries of every lane, loads ahead
template <int U, typename T>
__device__ __forceinline__ double small_four(const T *v, const uint16_t *c, const T *vec)
{
    T a[U], b[U];
    uint32_t ci[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        ci[q] = c[64 * q];
        a[q] = v[64 * q];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) b[q] = vec[ci[q]];
    double s = (double)a[0] * (double)b[0];
#pragma unroll
    for (int q = 1; q < U; ++q) s += (double)a[q] * (double)b[q];
    return s;
}

// a lane's k entries by fours into NS partial sums in turn, and their sum
template <int NS, typename T>
__device__ __forceinline__ double small_lane(int k, const T *v, const uint16_t *c, const T *vec)
{
    double acc[NS] = {};
    for (; k >= 4 * NS; k -= 4 * NS, v += 256 * NS, c += 256 * NS) {
#pragma unroll
        for (int q = 0; q < NS; ++q) acc[q] += small_four<4>(v + 256 * q, c + 256 * q, vec);
    }
#pragma unroll
    for (int q = 0; q < NS; ++q) {  // the rest: fewer than NS fours and a part of one
        if (k >= 4) {
            acc[q] += small_four<4>(v, c, vec);
            k -= 4, v += 256, c += 256;
        } else if (k > 0) {
            acc[q] += k == 3 ? small_four<3>(v, c, vec) : k == 2 ? small_four<2>(v, c, vec) : small_four<1>(v, c, vec);
            k = 0;
        }
    }
    if constexpr (NS == 4) return (acc[0] + acc[2]) + (acc[1] + acc[3]);
    if constexpr (NS == 2) return acc[0] + acc[1];
    return acc[0];
}

// v of the lane `n` places up, within rows of 16 lanes
template <int N>
__device__ __forceinline__ double lane_up(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x100 + N, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x100 + N, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// sum over groups of 2^lg lanes, valid in each group's first lane
__device__ __forceinline__ double lead_sum(double v, int lg)
{
    if (lg >= 6) v += __shfl_xor(v, 32);
    if (lg >= 5) v += __shfl_xor(v, 16);
    if (lg >= 4) v += lane_up<8>(v);
    if (lg >= 3) v += lane_up<4>(v);
    if (lg >= 2) v += lane_up<2>(v);
    if (lg >= 1) v += lane_up<1>(v);
    return v;
}

// The sums of the tasks' rows over the gathered vector; pre(row) runs in every
// lane ahead of the entries, fin(row, sum, pre) in each row's first lane.
template <typename T, typename P, typename F>
__device__ __forceinline__ void small_sweep(const SmallSlots<T> &o, const T *vec, P &&pre, F &&fin)
{
    const int wave = uniform_i(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int t = wave; t < o.ntask; t += SMALL_WG / 64) {
        const int4 tk = {o.task[4 * t], o.task[4 * t + 1], o.task[4 * t + 2], o.task[4 * t + 3]};
        const int lg = tk.z & 0xff;
        const int g = lane >> lg;
        const bool ok = g < tk.w;
        const int row = o.row[64 * t + (ok ? g : 0)];
        auto p = pre(row);
        const T *v = o.val + tk.x + lane;
        const uint16_t *c = o.col + tk.x + lane;
        double acc;
        switch (tk.z >> 8) {
            case 0: acc = small_lane<1>(tk.y, v, c, vec); break;
            case 1: acc = small_lane<2>(tk.y, v, c, vec); break;
            default: acc = small_lane<4>(tk.y, v, c, vec); break;
        }
        acc = lead_sum(acc, lg);
        if (ok && (lane & ((1 << lg) - 1)) == 0) fin(row, acc, p);
    }
}

__device__ __forceinline__ const __attribute__((address_space(4))) int32_t *small_tasks(const int4 *p)
{
    return (const __attribute__((address_space(4))) int32_t *)(uintptr_t)p;
}

template <typename T>
struct PreX {
    T x, c, l, u, xa, x0;
};
template <typename T>
struct PreY {
    T y, q, ya, y0;
};

template <typename X>
__device__ __forceinline__ X *lds_copy(X *&at, const X *src, int cnt)
{
    X *to = at;
    for (int i = threadIdx.x; i < cnt; i += SMALL_WG) to[i] = src[i];
    at += cnt;
    return to;
}

// LV: 1 K^T in LDS, 2 K too, 3 the updates' operands too.  MASK: the clips of step
// j go to masks.x / y(j0 + j); the lane that owns a row adds all of its bits.
template <typename T, bool AVG, bool MASK, int LV>
__device__ void small_run(const Dev &d, const SmallDev &sd, const InstInfo &in, const SmallInst &si, int j0, int count,
                          const Masks &masks)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int n = in.n, m = in.m, m1 = in.m1, tid = threadIdx.x;
    const InstState *st = d.st + blockIdx.x;
    const double tau = st->tau, sigma = st->sigma;
    T *gx = (T *)d.x + in.xoff, *gxb = (T *)d.xbar + in.xoff, *gxa = (T *)d.xavg + in.xoff;
    T *gy = (T *)d.y + in.yoff, *gya = (T *)d.yavg + in.yoff;
    const T *c = (const T *)d.c + in.xoff, *l = (const T *)d.l + in.xoff, *u = (const T *)d.u + in.xoff;
    const T *x0 = (const T *)d.x0 + in.xoff, *q = (const T *)d.q + in.yoff, *y0 = (const T *)d.y0 + in.yoff;
    SmallSlots<T> oT = {(const T *)sd.val[0] + si.slot0[0], sd.col[0] + si.slot0[0], nullptr,
                        small_tasks(sd.task[0] + si.task0[0]), si.ntask[0]};
    SmallSlots<T> oK = {(const T *)sd.val[1] + si.slot0[1], sd.col[1] + si.slot0[1], nullptr,
                        small_tasks(sd.task[1] + si.task0[1]), si.ntask[1]};

    // the layout small_bytes() counts
    double *wt = (double *)lds;
    if (AVG)
        for (int j = tid; j < count; j += SMALL_WG) wt[j] = 1.0 / (double)(st->t_inner + j0 + j + 1);
    T *at = (T *)(wt + SMALL_STEPS);
    T *x = lds_copy(at, (const T *)gx, n), *xb = at;
    at += n;
    T *xa = AVG ? lds_copy(at, (const T *)gxa, n) : nullptr;
    T *y = lds_copy(at, (const T *)gy, m);
    T *ya = AVG ? lds_copy(at, (const T *)gya, m) : nullptr;
    if (LV >= 1) oT.val = lds_copy(at, oT.val, si.nslot[0]);
    if (LV >= 2) oK.val = lds_copy(at, oK.val, si.nslot[1]);
    if (LV >= 3) {
        c = lds_copy(at, c, n);
        l = lds_copy(at, l, n);
        u = lds_copy(at, u, n);
        if (AVG) x0 = lds_copy(at, x0, n);
        q = lds_copy(at, q, m);
        if (AVG) y0 = lds_copy(at, y0, m);
    }
    uint16_t *at16 = (uint16_t *)at;
    oT.row = lds_copy(at16, sd.row[0] + 64 * (int64_t)si.task0[0], 64 * si.ntask[0]);
    oK.row = lds_copy(at16, sd.row[1] + 64 * (int64_t)si.task0[1], 64 * si.ntask[1]);
    if (LV >= 1) oT.col = lds_copy(at16, oT.col, si.nslot[0]);
    if (LV >= 2) oK.col = lds_copy(at16, oK.col, si.nslot[1]);
    __syncthreads();
    for (int j = 0; j < count; ++j) {
        const double w = AVG ? wt[j] : 0.0;
        const Mask mx = MASK ? masks.x(j0 + j) : Mask{}, my = MASK ? masks.y(j0 + j) : Mask{};
        small_sweep<T>(
            oT, y, [&](int r) -> PreX<T> { return {x[r], c[r], l[r], u[r], AVG ? xa[r] : T(0), AVG ? x0[r] : T(0)}; },
            [&](int r, double g, const PreX<T> &p) {
                const PrimalStep<T> s = primal_step<T>(p.x, g, p.c, p.l, p.u, tau);
                x[r] = s.x;
                xb[r] = s.xbar;
                if (AVG) xa[r] = average_step<T>(p.xa, s.x, p.x0, w);
                if (MASK) mask_put(mx.p, in.xoff + r, mx.sh, s.clip);
            });
        __syncthreads();
        small_sweep<T>(
            oK, xb, [&](int r) -> PreY<T> { return {y[r], q[r], AVG ? ya[r] : T(0), AVG ? y0[r] : T(0)}; },
            [&](int r, double a, const PreY<T> &p) {
                const DualStep<T> s = dual_step<T>(p.y, a, p.q, sigma, r < m1);
                y[r] = s.y;
                if (AVG) ya[r] = average_step<T>(p.ya, s.y, p.y0, w);
                if (MASK) mask_put(my.p, in.yoff + r, my.sh, s.pass);
            });
        __syncthreads();
    }
    for (int i = tid; i < n; i += SMALL_WG) {
        gx[i] = x[i];
        gxb[i] = xb[i];
        if (AVG) {
            gxa[i] = xa[i];
            ((T *)d.xam + in.xoff)[i] = (T)((double)x0[i] + (double)xa[i]);  // the average point, as k_avg_point
        }
    }
    for (int i = tid; i < m; i += SMALL_WG) {
        gy[i] = y[i];
        if (AVG) {
            gya[i] = ya[i];
            ((T *)d.yam + in.yoff)[i] = (T)((double)y0[i] + (double)ya[i]);
        }
    }
}

// Iterations j0 .. j0 + count - 1 (1 <= count <= SMALL_STEPS) of the current
// check period (MASK: of the steps of `masks`), one workgroup per instance.
template <typename T, bool AVG, bool MASK>
__global__ __launch_bounds__(SMALL_WG) void k_small(Dev d, SmallDev sd, int j0, int count, Masks masks)
{
    const SmallInst si = sd.inst[blockIdx.x];
    if (d.st[blockIdx.x].done) return;
    const InstInfo in = d.info[blockIdx.x];
    switch (si.level) {
        case 0: small_run<T, AVG, MASK, 0>(d, sd, in, si, j0, count, masks); break;
        case 1: small_run<T, AVG, MASK, 1>(d, sd, in, si, j0, count, masks); break;
        case 2: small_run<T, AVG, MASK, 2>(d, sd, in, si, j0, count, masks); break;
        default: small_run<T, AVG, MASK, 3>(d, sd, in, si, j0, count, masks); break;
    }
}

// values and columns of the slots from the scaled operator: slot s holds the
// instance's entry src[s], or with a zero value (padding) the entry ~src[s]
template <typename T>
__global__ void k_small_fill(OpDev op, const SmallInst *inst, int o, const InstInfo *info, const int32_t *src, T *val,
                             uint16_t *col)
{
    const SmallInst si = inst[blockIdx.x];
    const int64_t roff = o == 0 ? info[blockIdx.x].xoff : info[blockIdx.x].yoff;
    const int64_t coff = o == 0 ? info[blockIdx.x].yoff : info[blockIdx.x].xoff;
    const int64_t e0 = op.rp[roff];
    for (int s = threadIdx.x; s < si.nslot[o]; s += SMALL_WG) {
        const int32_t e = src[si.slot0[o] + s];
        val[si.slot0[o] + s] = e >= 0 ? op_vals<T>(op)[e0 + e] : T(0);
        col[si.slot0[o] + s] = (uint16_t)(op.ci[e0 + (e >= 0 ? e : ~e)] - coff);
    }
}

}  // namespace

template <typename T>
void launch_small(const Dev &d, const SmallDev &sd, int j0, int count, int avg, hipStream_t s)
{
    for (int j = 0; j < count; j += SMALL_STEPS) {
        const int k = count - j < SMALL_STEPS ? count - j : SMALL_STEPS;
        if (avg)
            hipLaunchKernelGGL((k_small<T, true, false>), dim3(d.batch), dim3(SMALL_WG), sd.lds, s, d, sd, j0 + j, k, Masks{});
        else
            hipLaunchKernelGGL((k_small<T, false, false>), dim3(d.batch), dim3(SMALL_WG), sd.lds, s, d, sd, j0 + j, k, Masks{});
    }
}

// Steps t0 .. t0 + count - 1 of `masks`, which receives their clips.
template <typename T>
void launch_small_masked(const Dev &d, const SmallDev &sd, const Masks &masks, int64_t t0, int count, hipStream_t s)
{
    for (int j = 0; j < count; j += SMALL_STEPS) {
        const int k = count - j < SMALL_STEPS ? count - j : SMALL_STEPS;
        hipLaunchKernelGGL((k_small<T, false, true>), dim3(d.batch), dim3(SMALL_WG), sd.lds, s, d, sd, (int)t0 + j, k, masks);
    }
}

template <typename T>
void launch_small_fill(const Dev &d, const SmallDev &sd, hipStream_t s)
{
    for (int o = 0; o < 2; ++o)
        hipLaunchKernelGGL(k_small_fill<T>, dim3(d.batch), dim3(SMALL_WG), 0, s, o == 0 ? d.Kt : d.K, sd.inst, o, d.info,
                           sd.src[o], (T *)sd.val[o], sd.col[o]);
}

// lets the kernels take a CU's whole LDS on the current device (the limit is the
// kernel's, not a handle's: the same for handles of all sizes)
hipError_t small_prepare()
{
    const void *k[6] = {(const void *)k_small<float, true, false>,  (const void *)k_small<float, false, false>,
                        (const void *)k_small<float, false, true>,  (const void *)k_small<double, true, false>,
                        (const void *)k_small<double, false, false>, (const void *)k_small<double, false, true>};
    for (const void *f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SMALL_LDS);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

#define SMALL_INST(T)                                                                                              \
    template void launch_small<T>(const Dev &, const SmallDev &, int, int, int, hipStream_t); \
    template void launch_small_masked<T>(const Dev &, const SmallDev &, const Masks &, int64_t, int, hipStream_t); \
    template void launch_small_fill<T>(const Dev &, const SmallDev &, hipStream_t);
SMALL_INST(float)
SMALL_INST(double)

}  // namespace pdhg
