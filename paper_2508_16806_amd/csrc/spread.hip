// spread.hip -- sweeps over vectors too long for the L2s, in two passes.
//
// The row-binned sweeps issue one L2 request per matrix entry; over columns
// without locality in a vector of several MB most of them miss the 4 MB L2 of
// their XCD as well (94-148 G gathers/s at 54M nonzeros, against 165-280 out of
// L2).  Rows that meet every column tile less than once cannot take the vector
// through LDS either (tile.hip).  So the gather and the sums are split, and both
// stream:
//   1. k_spread: the entries ordered by column tile (64 KB of the vector, copied
//      to LDS), 16-bit columns within the tile; the gathered values are written
//      to a buffer in that order.
//   2. k_spread_primal / _dual: a workgroup per window (a run of rows with up to
//      SPREAD_BYTES of values).  The window's values lie in one run per tile in
//      the buffer, are copied to LDS, and the rows are summed from there in the
//      order of the row-binned sweep through a 16-bit place per entry, so the
//      sums are the same to the bit.  Then the update, one leader per row.
// 16 bytes an entry in FP32 (2 column, 4 + 4 value written and read back, 2 place,
// 4 matrix) against a 64-byte line per entry: bound by memory now, 54M nonzeros
// take 77 us (4.2 TB/s) and 151-162 us (3.3-3.5 TB/s), 223-236 us a sweep where
// the row-binned sweeps took 379 (vector of 4 MB) and 595 (8 MB).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "sweep.h"

namespace pdhg {
namespace {

// n elements at LDS place `to` from src, 4 bytes a lane, by one wavefront
template <typename T>
__device__ __forceinline__ void wave_copy(const T *src, T *to, int n)
{
    const int words = n * (int)(sizeof(T) / 4), lane = threadIdx.x & 63;
    const uint32_t *from = (const uint32_t *)src;
    for (int k = 0; k < words; k += 64)
        if (k + lane < words)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) unsigned int *)(from + k + lane),
                                             (__attribute__((address_space(3))) unsigned int *)((uint32_t *)to + k), 4, 0, 0);
}

// Pass 1.  Every workgroup takes an equal run of the entries in tile order and
// the tiles (1.2 on average at two workgroups per CU) they lie in.
template <typename T, int OP>
__global__ __launch_bounds__(SPREAD_WG, 8) void k_spread(Dev d, SpreadOp op, const T *__restrict__ v)
{
    constexpr int WIDTH = SPREAD_TILE / (int)sizeof(T);
    __shared__ __align__(16) T tile[WIDTH];
    if (d.act_cnt[OP == 0 ? 1 : 0] == 0) return;
    const uint16_t *__restrict__ idx = op.idx;
    T *__restrict__ g = (T *)op.g;
    const int tid = threadIdx.x;
    const uint32_t per = ((op.n + gridDim.x - 1) / gridDim.x + 7) & ~7u;
    if ((uint64_t)blockIdx.x * per >= op.n) return;
    uint32_t k0 = blockIdx.x * per;
    const uint32_t k1 = op.n - k0 < per ? op.n : k0 + per;
    // the tile of entry k0: the last one that starts at or before it
    int lo = 0, hi = op.nt;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (op.tb[mid] <= k0)
            lo = mid;
        else
            hi = mid;
    }
    for (int t = lo; t < op.nt && k0 < k1; ++t) {
        const uint32_t e = min(k1, op.tb[t + 1]);
        if (e <= k0) continue;
        const int c0 = t * WIDTH, bytes = min(WIDTH, op.ncol - c0) * (int)sizeof(T);
        __syncthreads();
        // whole 16-byte lines: the vector starts on one and is padded
        const uint4 *from = (const uint4 *)(v + c0);
        for (int i = tid & ~63; i < (bytes + 15) / 16; i += SPREAD_WG)
            if (i + (tid & 63) < (bytes + 15) / 16)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) unsigned int *)(from + i + (tid & 63)),
                    (__attribute__((address_space(3))) unsigned int *)((uint4 *)tile + i), 16, 0, 0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        // eight entries a lane; the ends one by one
        const uint32_t a0 = min(e, (k0 + 7) & ~7u), a1 = max(a0, e & ~7u);
        if (tid < 8 && k0 + tid < a0) g[k0 + tid] = tile[idx[k0 + tid]];
        if (tid >= 8 && tid < 16 && a1 + (tid - 8) < e) g[a1 + (tid - 8)] = tile[idx[a1 + (tid - 8)]];
        auto eight = [&](uint32_t k, uint4 c) {
            const uint32_t w[4] = {c.x, c.y, c.z, c.w};
            T r[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                r[2 * i] = tile[w[i] & 0xffff];
                r[2 * i + 1] = tile[w[i] >> 16];
            }
            uint4 *to = (uint4 *)(g + k);
#pragma unroll
            for (int i = 0; i < (int)sizeof(T) / 2; ++i) to[i] = ((const uint4 *)r)[i];
        };
        uint32_t k = a0 + 8 * tid;
        for (; k + 8 * SPREAD_WG < a1; k += 16 * SPREAD_WG) {
            const uint4 c0q = *(const uint4 *)(idx + k), c1q = *(const uint4 *)(idx + k + 8 * SPREAD_WG);
            eight(k, c0q);
            eight(k + 8 * SPREAD_WG, c1q);
        }
        if (k < a1) eight(k, *(const uint4 *)(idx + k));
        k0 = e;
    }
}

// Pass 2: pre(row) loads the operands of a row ahead of its sum and returns the
// update as a function of that sum.
template <typename T, typename MV, typename Pre>
__device__ __forceinline__ void spread_rows(const OpDev &op, const SpreadOp &so, Pre &&pre)
{
    __shared__ __align__(16) T win[SPREAD_BYTES / sizeof(T)];
    __shared__ double part[SPREAD_WG / 64];
    const int tid = threadIdx.x, wave = uniform_i(tid >> 6), lane = tid & 63;
    const int4 b = so.win[blockIdx.x];
    const int nt = so.nt;
    {
        const uint32_t *start = so.start + (size_t)blockIdx.x * nt, *lofs = so.lofs + (size_t)blockIdx.x * (nt + 1);
        const int t = wave + 16 * lane;
        uint32_t s = 0, l = 0, n = 0;
        if (t < nt) {
            s = start[t];
            l = lofs[t];
            n = lofs[t + 1] - l;
        }
        const T *g = (const T *)so.g;
        for (int i = 0; wave + 16 * i < nt; ++i)
            wave_copy(g + (uint32_t)__builtin_amdgcn_readlane((int)s, i), win + __builtin_amdgcn_readlane((int)l, i),
                      __builtin_amdgcn_readlane((int)n, i));
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int64_t *__restrict__ rp = op.rp + b.x;
    const int64_t p0 = rp[0];
    const uint16_t *__restrict__ place = so.place + p0;
    const MV *__restrict__ va = op_vals<MV>(op) + p0;
    const int lg = b.z, L = 1 << lg, G = SPREAD_WG >> lg, gl = tid & (L - 1);
    for (int r0 = 0; r0 < b.y; r0 += G) {
        const int r = r0 + (tid >> lg);
        const bool ok = r < b.y;
        const int rr = ok ? r : b.y - 1;
        const uint32_t o0 = (uint32_t)(rp[rr] - p0);
        const uint32_t o1 = ok ? (uint32_t)(rp[rr + 1] - p0) : o0;
        auto update = pre((int64_t)b.x + rr);
        double acc = 0.0;
        for (uint32_t p = o0 + gl; p < o1; p += 4 * L) {
            uint32_t at[4];
            MV a[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t q = p + k * L < o1 ? p + k * L : p;
                at[k] = ldo(place, q);
                a[k] = ldo(va, q);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double v = p + k * L < o1 ? (double)a[k] : 0.0;
                acc += v * (double)win[at[k]];
            }
        }
        for (int off = min(L, 64) >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
        if (lg > 6) {
            if (lane == 0) part[wave] = acc;
            __syncthreads();
            const double *q = part + (wave & ~3);
            acc = (q[0] + q[1]) + (q[2] + q[3]);
            __syncthreads();
        }
        if (gl == 0 && ok) update(acc);
    }
}

template <typename T, int AVG, int MASK>
__global__ __launch_bounds__(SPREAD_WG, 8) void k_spread_primal(Dev d, SpreadOp so, int j_in_chunk, Mask mask)
{
    if (d.act_cnt[1] == 0) return;
    T *__restrict__ x = (T *)d.x;
    T *__restrict__ xb = (T *)d.xbar;
    T *__restrict__ xa = (T *)d.xavg;
    const double tau = d.st->tau;
    const double w = AVG ? 1.0 / (double)(d.st->t_inner + j_in_chunk + 1) : 0.0;
    spread_rows<T, T>(d.Kt, so, [&](int64_t j) {
        const T v_x = x[j], v_c = ((const T *)d.c)[j], v_l = ((const T *)d.l)[j], v_u = ((const T *)d.u)[j];
        const T v_a = AVG ? xa[j] : T(0), v_0 = AVG ? ((const T *)d.x0)[j] : T(0);
        return [=](double g) {
            const PrimalStep<T> p = primal_step<T>(v_x, g, v_c, v_l, v_u, tau);
            x[j] = p.x;
            xb[j] = p.xbar;
            if (AVG) xa[j] = average_step<T>(v_a, p.x, v_0, w);
            if (MASK) mask_put(mask.p, j, mask.sh, p.clip);
        };
    });
}

template <typename T, int AVG, int MASK>
__global__ __launch_bounds__(SPREAD_WG, 8) void k_spread_dual(Dev d, SpreadOp so, int j_in_chunk, int64_t m1,
                                                             Mask mask)
{
    if (d.act_cnt[0] == 0) return;
    T *__restrict__ y = (T *)d.y;
    T *__restrict__ ya = (T *)d.yavg;
    const double sigma = d.st->sigma;
    const double w = AVG ? 1.0 / (double)(d.st->t_inner + j_in_chunk + 1) : 0.0;
    spread_rows<T, T>(d.K, so, [&](int64_t i) {
        const T v_y = y[i], v_q = ((const T *)d.q)[i];
        const T v_a = AVG ? ya[i] : T(0), v_0 = AVG ? ((const T *)d.y0)[i] : T(0);
        return [=](double r) {
            const DualStep<T> p = dual_step<T>(v_y, r, v_q, sigma, i < m1);
            y[i] = p.y;
            if (AVG) ya[i] = average_step<T>(v_a, p.y, v_0, w);
            if (MASK) mask_put(mask.p, i, mask.sh, p.pass);
        };
    });
}

// The FP64 products a check needs (k_check's sums to the bit: the same values in
// the same order), one per row.
template <typename T, int OP>
__global__ __launch_bounds__(SPREAD_WG, 8) void k_spread_products(Dev d, SpreadOp so, double *__restrict__ out)
{
    if (d.act_cnt[OP == 0 ? 1 : 0] == 0) return;
    spread_rows<T, double>(OP == 0 ? d.Kt : d.K, so, [&](int64_t r) { return [=](double g) { out[r] = g; }; });
}

// The layout, from the CSR operator: entries per window and tile with their
// places in the window; where each tile's runs start; then columns and places.
// The order within a run is whatever the atomics give: no sum depends on it.
__global__ __launch_bounds__(SPREAD_WG) void k_spread_count(OpDev op, SpreadOp so, int width)
{
    __shared__ uint32_t cnt[SPREAD_TILES];
    const int tid = threadIdx.x;
    const int4 b = so.win[blockIdx.x];
    cnt[tid] = 0;
    __syncthreads();
    const int64_t p1 = op.rp[b.x + b.y];
    for (int64_t p = op.rp[b.x] + tid; p < p1; p += SPREAD_WG) atomicAdd(&cnt[op.ci[p] / width], 1u);
    __syncthreads();
    const uint32_t n = cnt[tid];
    for (int off = 1; off < SPREAD_TILES; off <<= 1) {
        const uint32_t a = tid >= off ? cnt[tid - off] : 0;
        __syncthreads();
        cnt[tid] += a;
        __syncthreads();
    }
    uint32_t *lofs = so.lofs + (size_t)blockIdx.x * (so.nt + 1);
    if (tid < so.nt) {
        lofs[tid] = cnt[tid] - n;
        if (tid == so.nt - 1) lofs[so.nt] = cnt[tid];
    }
}

// one workgroup per tile: its runs' starts within the tile
__global__ __launch_bounds__(SPREAD_WG) void k_spread_scan(SpreadOp so)
{
    __shared__ uint32_t s[SPREAD_WG];
    const int tid = threadIdx.x, t = blockIdx.x;
    uint32_t carry = 0;
    for (int w0 = 0; w0 < so.nwin; w0 += SPREAD_WG) {
        const int w = w0 + tid;
        const uint32_t *lofs = so.lofs + (size_t)w * (so.nt + 1) + t;
        const uint32_t n = w < so.nwin ? lofs[1] - lofs[0] : 0;
        s[tid] = n;
        __syncthreads();
        for (int off = 1; off < SPREAD_WG; off <<= 1) {
            const uint32_t a = tid >= off ? s[tid - off] : 0;
            __syncthreads();
            s[tid] += a;
            __syncthreads();
        }
        if (w < so.nwin) so.start[(size_t)w * so.nt + t] = carry + s[tid] - n;
        carry += s[SPREAD_WG - 1];
        __syncthreads();
    }
    if (tid == 0) so.tb[t + 1] = carry;
}

// one workgroup: the tiles' starts from their sizes
__global__ __launch_bounds__(SPREAD_WG) void k_spread_base(SpreadOp so)
{
    __shared__ uint32_t s[SPREAD_WG];
    const int tid = threadIdx.x;
    s[tid] = tid < so.nt ? so.tb[tid + 1] : 0;
    __syncthreads();
    for (int off = 1; off < SPREAD_WG; off <<= 1) {
        const uint32_t a = tid >= off ? s[tid - off] : 0;
        __syncthreads();
        s[tid] += a;
        __syncthreads();
    }
    if (tid < so.nt) so.tb[tid + 1] = s[tid];
    if (tid == 0) so.tb[0] = 0;
}

__global__ __launch_bounds__(SPREAD_WG) void k_spread_fill(OpDev op, SpreadOp so, int width)
{
    __shared__ uint32_t at[SPREAD_TILES], first[SPREAD_TILES], run[SPREAD_TILES];
    const int tid = threadIdx.x;
    const int4 b = so.win[blockIdx.x];
    if (tid < so.nt) {
        const size_t k = (size_t)blockIdx.x * so.nt + tid;
        first[tid] = at[tid] = so.lofs[(size_t)blockIdx.x * (so.nt + 1) + tid];
        run[tid] = so.start[k] + so.tb[tid];
        so.start[k] = run[tid];
    }
    __syncthreads();
    const int64_t p1 = op.rp[b.x + b.y];
    for (int64_t p = op.rp[b.x] + tid; p < p1; p += SPREAD_WG) {
        const int c = op.ci[p], t = c / width;
        const uint32_t k = atomicAdd(&at[t], 1u);
        so.place[p] = (uint16_t)k;
        so.idx[run[t] + (k - first[t])] = (uint16_t)(c - t * width);
    }
}

}  // namespace

template <typename T>
void launch_spread_primal(const Dev &d, const SpreadOp &so, int j, int avg, Mask mask, hipStream_t s)
{
    const dim3 g(so.nwin), wg(SPREAD_WG);
    hipLaunchKernelGGL((k_spread<T, 0>), dim3(SPREAD_GRID), wg, 0, s, d, so, (const T *)d.y);
    if (mask.p)
        hipLaunchKernelGGL((k_spread_primal<T, 0, 1>), g, wg, 0, s, d, so, j, mask);
    else if (avg)
        hipLaunchKernelGGL((k_spread_primal<T, 1, 0>), g, wg, 0, s, d, so, j, mask);
    else
        hipLaunchKernelGGL((k_spread_primal<T, 0, 0>), g, wg, 0, s, d, so, j, mask);
}

template <typename T>
void launch_spread_dual(const Dev &d, const SpreadOp &so, int j, int avg, int64_t m1, Mask mask, hipStream_t s)
{
    const dim3 g(so.nwin), wg(SPREAD_WG);
    hipLaunchKernelGGL((k_spread<T, 1>), dim3(SPREAD_GRID), wg, 0, s, d, so, (const T *)d.xbar);
    if (mask.p)
        hipLaunchKernelGGL((k_spread_dual<T, 0, 1>), g, wg, 0, s, d, so, j, m1, mask);
    else if (avg)
        hipLaunchKernelGGL((k_spread_dual<T, 1, 0>), g, wg, 0, s, d, so, j, m1, mask);
    else
        hipLaunchKernelGGL((k_spread_dual<T, 0, 0>), g, wg, 0, s, d, so, j, m1, mask);
}

template <typename T>
void launch_spread_products(const Dev &d, const SpreadOp &so, int onK, const void *v, double *out, hipStream_t s)
{
    const dim3 g(so.nwin), wg(SPREAD_WG);
    if (onK) {
        hipLaunchKernelGGL((k_spread<T, 1>), dim3(SPREAD_GRID), wg, 0, s, d, so, (const T *)v);
        hipLaunchKernelGGL((k_spread_products<T, 1>), g, wg, 0, s, d, so, out);
    } else {
        hipLaunchKernelGGL((k_spread<T, 0>), dim3(SPREAD_GRID), wg, 0, s, d, so, (const T *)v);
        hipLaunchKernelGGL((k_spread_products<T, 0>), g, wg, 0, s, d, so, out);
    }
}

template <typename T>
void launch_spread_build(const OpDev &op, const SpreadOp &so, hipStream_t s)
{
    const int width = SPREAD_TILE / (int)sizeof(T);
    hipLaunchKernelGGL(k_spread_count, dim3(so.nwin), dim3(SPREAD_WG), 0, s, op, so, width);
    hipLaunchKernelGGL(k_spread_scan, dim3(so.nt), dim3(SPREAD_WG), 0, s, so);
    hipLaunchKernelGGL(k_spread_base, dim3(1), dim3(SPREAD_WG), 0, s, so);
    hipLaunchKernelGGL(k_spread_fill, dim3(so.nwin), dim3(SPREAD_WG), 0, s, op, so, width);
}

#define SPREAD_INST(T)                                                                                      \
    template void launch_spread_primal<T>(const Dev &, const SpreadOp &, int, int, Mask, hipStream_t);       \
    template void launch_spread_dual<T>(const Dev &, const SpreadOp &, int, int, int64_t, Mask, hipStream_t); \
    template void launch_spread_products<T>(const Dev &, const SpreadOp &, int, const void *, double *, hipStream_t); \
    template void launch_spread_build<T>(const OpDev &, const SpreadOp &, hipStream_t);
SPREAD_INST(float)
SPREAD_INST(double)

}  // namespace pdhg
