// tile.hip -- sweeps that gather from LDS ("tiles").
//
// The row-binned sweeps issue one L2 request per matrix entry: over columns
// without locality that request rate (165-280 G/s on the chip, falling with the
// matrix' size), not the matrix stream, is what bounds them.  Here one 1024-lane
// workgroup per CU owns a run of rows and takes the gathered vector through LDS
// in tiles of up to 128 KB: it copies a tile to LDS, walks its rows' entries that
// fall into the tile, and goes on to the next one; the rows' FP64 sums stay in
// LDS, and after the last tile one lane per row makes the update with coalesced
// operands.  (Half the width in two buffers, the next tile on its way meanwhile,
// was slower: 14.5 / 15.9 us against 11.5 / 12.3 at 5M nonzeros, since a row's
// shorter pieces leave fewer loads in flight.)
//
// Layout (built by k_tile_build from the CSR images): per block, tile by tile
// and row by row, the entries of the row in the tile, padded to fours ("quads")
// so that a lane loads four values and four 16-bit columns at once: 6 bytes an
// entry in FP32 instead of 8, 10 instead of 12 in FP64.
//
// 256 blocks (one per CU) measured best at 31M nonzeros (us, 256 / 512 / 1,024:
// 36 / 40 / 56): more blocks load the vector more often.  2^lg lanes per row such
// that a lane has 2 to 4 quads (tile_lg()).  Measured, us per sweep (row bins /
// here): FP32, 50,000 rows over 125,000 columns, 31M nonzeros 190 / 52; its
// transpose 195 / 46.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "sweep.h"

namespace pdhg {
namespace {

template <typename V>
struct Quad;
template <>
struct Quad<float> {
    float4 v;
    __device__ __forceinline__ void load(const float *p, uint32_t q) { v = ldo((const float4 *)p, q); }
};
template <>
struct Quad<double> {
    double4 v;
    __device__ __forceinline__ void load(const double *p, uint32_t q)
    {
        const double2 a = ldo((const double2 *)p, 2 * q), b = ldo((const double2 *)p, 2 * q + 1);
        v = make_double4(a.x, a.y, b.x, b.y);
    }
};

// LDS of a block: the rows' sums, the rows' quad ranges, the tile
extern __shared__ __align__(16) unsigned char tile_raw[];
__device__ __forceinline__ double *tile_sum() { return (double *)tile_raw; }
__device__ __forceinline__ uint32_t *tile_ptr() { return (uint32_t *)(tile_raw + 8 * TILE_ROWS); }
__device__ __forceinline__ unsigned char *tile_vec() { return tile_raw + TILE_LDS - TILE_BYTES; }

// n elements of src straight to LDS (no registers in between), from the 16-byte
// line that holds the first one on: an instance's part of a batch's vector starts
// anywhere; the vectors are 256-byte aligned and padded.  Returns the place of
// src[0] in LDS.  The caller waits for its loads and for the workgroup.
template <int W, typename GV>
__device__ __forceinline__ const GV *tile_copy(const GV *src, int n)
{
    const int skip = (int)(((uintptr_t)src & 15) / sizeof(GV));
    const int cnt = ((skip + n) * (int)sizeof(GV) + 15) / 16, lane = threadIdx.x & 63;
    const uint4 *from = (const uint4 *)(src - skip);
    for (int i = uniform_i((int)threadIdx.x & ~63); i < cnt; i += W)
        if (i + lane < cnt)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) unsigned int *)(from + i + lane),
                (__attribute__((address_space(3))) unsigned int *)(tile_vec() + 16 * i), 16, 0, 0);
    return (const GV *)tile_vec() + skip;
}

// U quads of one lane: q, q + 2^lg, ... below q1
template <typename MV, int U>
struct TileRegs {
    Quad<MV> a[U];
    uint2 c[U];
    __device__ __forceinline__ void load(const MV *va, const uint2 *ix, uint32_t q, uint32_t q1, int lg)
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t p = q + (uint32_t)(u << lg);
            p = p < q1 ? p : q;
            a[u].load(va, p);
            c[u] = ldo(ix, p);
        }
    }
    template <typename GV>
    __device__ __forceinline__ double dot(double acc, const GV *vec, uint32_t q, uint32_t q1, int lg) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double x0 = (double)vec[c[u].x & 0xffff], x1 = (double)vec[c[u].x >> 16];
            const double x2 = (double)vec[c[u].y & 0xffff], x3 = (double)vec[c[u].y >> 16];
            double s = (double)a[u].v.x * x0;
            s += (double)a[u].v.y * x1;
            s += (double)a[u].v.z * x2;
            s += (double)a[u].v.w * x3;
            acc += q + (uint32_t)(u << lg) < q1 ? s : 0.0;
        }
        return acc;
    }
};

// The same sums with gathers from global memory, for blocks whose entries are
// too few to pay for the tile: no copy, no barrier before the end.
template <int W, typename MV, typename GV>
__device__ __forceinline__ void tile_dots_direct(const TileOp &op, const MV *val, const TileBlk &b, const GV *vec)
{
    constexpr int U = 4;
    const int tid = threadIdx.x;
    const MV *va = val + 4 * b.q0;
    const uint2 *ix = op.idx + b.q0;
    double *sum = tile_sum();
    int lg = b.lg0, end = b.end0, r = tid >> lg;
    for (int k = 0;;) {
        const int lane = tid & ((1 << lg) - 1);
        for (; r < end; r += W >> lg) {
            const uint32_t *sp = op.sp + b.sp0;
            const GV *x = vec + b.coff;
            double part = 0.0;
            for (int t = 0; t < b.ntile; ++t, sp += b.nrows, x += b.width) {
                const uint32_t q1 = ldo(sp, (uint32_t)r + 1);
                double acc = 0.0;
                for (uint32_t q = ldo(sp, (uint32_t)r) + lane; q < q1; q += U << lg) {
                    TileRegs<MV, U> w;
                    w.load(va, ix, q, q1, lg);
                    acc = w.dot(acc, x, q, q1, lg);
                }
                for (int off = 1 << lg >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
                part += acc;
            }
            if (lane == 0) sum[r] = part;
        }
        if (++k == b.nrun) break;
        const int4 run = op.run[b.run0 + k];
        lg = run.z, end = run.y, r = run.x + (tid >> lg);
    }
    __syncthreads();
}

// The row sums of block b over the gathered vector into tile_sum(), by a
// workgroup of W lanes.  A workgroup barrier ends it.  The quads of each lane's
// first row are on their way while the tile is copied.
template <int W, typename MV, typename GV>
__device__ __forceinline__ void tile_dots(const TileOp &op, const MV *val, const TileBlk &b, const GV *vec)
{
    if constexpr (W < TILE_WG) {
        tile_dots_direct<W>(op, val, b, vec);
        return;
    }
    constexpr int U = 2;
    const int tid = threadIdx.x;
    const MV *va = val + 4 * b.q0;
    const uint2 *ix = op.idx + b.q0;
    const uint32_t *sp = op.sp + b.sp0;
    double *sum = tile_sum();
    uint32_t *ptr = tile_ptr();
    vec += b.coff;
    for (int r = tid; r < b.nrows; r += W) sum[r] = 0.0;
    for (int t = 0; t < b.ntile; ++t, sp += b.nrows, vec += b.width) {
        if (t > 0) __syncthreads();
        TileRegs<MV, U> w;
        int lg = b.lg0, end = b.end0, lane = tid & ((1 << lg) - 1), r = tid >> lg;
        uint32_t q = 0, q1 = 0;
        if (r < end) {
            q = ldo(sp, (uint32_t)r) + lane;
            q1 = ldo(sp, (uint32_t)r + 1);
        }
        const GV *x = tile_copy<W>(vec, min(b.width, b.ncol - t * b.width));
        if (q < q1) w.load(va, ix, q, q1, lg);
        for (int i = tid; i <= b.nrows; i += W) ptr[i] = ldo(sp, (uint32_t)i);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the lane's part of the tile is in LDS
        __syncthreads();
        for (int k = 0;;) {
            while (r < end) {
                double acc = 0.0;
                while (q < q1) {
                    acc = w.dot(acc, x, q, q1, lg);
                    q += U << lg;
                    if (q < q1) w.load(va, ix, q, q1, lg);
                }
                for (int off = 1 << lg >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
                if (lane == 0) sum[r] += acc;
                r += W >> lg;
                if (r >= end) break;
                q = ptr[r] + lane;
                q1 = ptr[r + 1];
                if (q < q1) w.load(va, ix, q, q1, lg);
            }
            if (++k == b.nrun) break;
            const int4 run = op.run[b.run0 + k];  // {first row, end row, lanes_log2, 0}
            lg = run.z, end = run.y, lane = tid & ((1 << lg) - 1), r = run.x + (tid >> lg);
            if (r >= end) continue;
            q = ptr[r] + lane;
            q1 = ptr[r + 1];
            if (q < q1) w.load(va, ix, q, q1, lg);
        }
    }
    __syncthreads();
}

// a block's descriptor in scalar registers
__device__ __forceinline__ TileBlk tile_blk(const TileBlk *p)
{
    constexpr int W = sizeof(TileBlk) / 4;
    union {
        TileBlk b;
        int w[W];
    } u;
    const int *src = (const int *)p;
#pragma unroll
    for (int k = 0; k < W; ++k) u.w[k] = uniform_i(src[k]);
    return u.b;
}

// f(block) for the blocks of the running instances
template <typename F>
__device__ __forceinline__ void tile_blocks(const TileOp &op, const int32_t *cntp, F &&f)
{
    // the block and its list entry are loaded beside the count: with every block
    // active the list is the identity (the grid has at most nblk workgroups)
    TileBlk b = tile_blk(op.blk + blockIdx.x);
    int next = uniform_i(op.act[blockIdx.x]);
    const int cnt = *cntp;
    const bool full = cnt == op.nblk;
    for (int it = blockIdx.x; it < cnt; it += gridDim.x) {
        if (it >= (int)gridDim.x) next = uniform_i(op.act[it]);
        if (!full || it >= (int)gridDim.x) b = tile_blk(op.blk + (full ? it : next));
        f(b);
        __syncthreads();
    }
}

template <int W, typename T, int AVG, int MASK>
__global__ __launch_bounds__(W) void k_primal_tile(Dev d, TileOp op, int j_in_chunk, Mask mask)
{
    T *__restrict__ x = (T *)d.x;
    T *__restrict__ xb = (T *)d.xbar;
    T *__restrict__ xa = (T *)d.xavg;
    const T *__restrict__ x0 = (const T *)d.x0;
    const T *__restrict__ c = (const T *)d.c;
    const T *__restrict__ l = (const T *)d.l;
    const T *__restrict__ u = (const T *)d.u;
    tile_blocks(op, d.act_cnt + 3, [&](const TileBlk &b) {
        const InstState *st = d.st + b.inst;
        const double tau = st->tau;
        const double w = AVG ? 1.0 / (double)(st->t_inner + j_in_chunk + 1) : 0.0;
        // the operands of the lane's first row are loaded ahead of the sums
        const uint32_t j0 = (uint32_t)(b.row0 + min((int)threadIdx.x, b.nrows - 1));
        T v_x = ldo(x, j0), v_c = ldo(c, j0), v_l = ldo(l, j0), v_u = ldo(u, j0);
        T v_a = AVG ? ldo(xa, j0) : T(0), v_0 = AVG ? ldo(x0, j0) : T(0);
        tile_dots<W, T, T>(op, (const T *)op.val, b, (const T *)d.y);
        for (int r = threadIdx.x; r < b.nrows; r += W) {
            const int64_t j = b.row0 + r;
            if (r >= W) {
                v_x = x[j], v_c = c[j], v_l = l[j], v_u = u[j];
                if (AVG) v_a = xa[j], v_0 = x0[j];
            }
            const PrimalStep<T> p = primal_step<T>(v_x, tile_sum()[r], v_c, v_l, v_u, tau);
            x[j] = p.x;
            xb[j] = p.xbar;
            if (AVG) xa[j] = average_step<T>(v_a, p.x, v_0, w);
            if (MASK) mask_put(mask.p, j, mask.sh, p.clip);
        }
    });
}

template <int W, typename T, int AVG, int MASK>
__global__ __launch_bounds__(W) void k_dual_tile(Dev d, TileOp op, int j_in_chunk, Mask mask)
{
    T *__restrict__ y = (T *)d.y;
    T *__restrict__ ya = (T *)d.yavg;
    const T *__restrict__ y0 = (const T *)d.y0;
    const T *__restrict__ q = (const T *)d.q;
    tile_blocks(op, d.act_cnt + 2, [&](const TileBlk &b) {
        const InstState *st = d.st + b.inst;
        const double sigma = st->sigma;
        const double w = AVG ? 1.0 / (double)(st->t_inner + j_in_chunk + 1) : 0.0;
        const uint32_t i0 = (uint32_t)(b.row0 + min((int)threadIdx.x, b.nrows - 1));
        T v_y = ldo(y, i0), v_q = ldo(q, i0), v_a = AVG ? ldo(ya, i0) : T(0), v_0 = AVG ? ldo(y0, i0) : T(0);
        tile_dots<W, T, T>(op, (const T *)op.val, b, (const T *)d.xbar);
        for (int r = threadIdx.x; r < b.nrows; r += W) {
            const int64_t i = b.row0 + r;
            if (r >= W) {
                v_y = y[i], v_q = q[i];
                if (AVG) v_a = ya[i], v_0 = y0[i];
            }
            const DualStep<T> p = dual_step<T>(v_y, tile_sum()[r], v_q, sigma, r < b.nineq);
            y[i] = p.y;
            if (AVG) ya[i] = average_step<T>(v_a, p.y, v_0, w);
            if (MASK) mask_put(mask.p, i, mask.sh, p.pass);
        }
    });
}

// The layout of one block per workgroup, from its rows of the CSR operator: the
// entries of each tile and row counted, the quad ranges by a scan over the
// block, then the entries placed in row order.
template <typename T>
__global__ __launch_bounds__(TILE_WG) void k_tile_build(OpDev op, TileOp to)
{
    constexpr int NW = TILE_WG / 64;
    __shared__ uint32_t cnt[TILE_SEGS + 1];
    __shared__ uint32_t scan[TILE_WG];
    const TileBlk b = to.blk[blockIdx.x];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nseg = b.nrows * b.ntile;
    for (int i = tid; i <= nseg; i += TILE_WG) cnt[i] = 0;
    __syncthreads();
    // tile and column within it
    auto split = [&](int32_t c, int &loc) {
        int t = 0;
        for (int k = 1; k < b.ntile; ++k) t += c >= k * b.width;
        loc = c - t * b.width;
        return t;
    };
    auto seg = [&](int r, int t) { return t * b.nrows + r; };
    for (int r = wave; r < b.nrows; r += NW) {
        const int64_t p0 = op.rp[b.row0 + r], p1 = op.rp[b.row0 + r + 1];
        for (int64_t p = p0 + lane; p < p1; p += 64) {
            int loc;
            const int s = split((int32_t)(op.ci[p] - b.coff), loc);
            atomicAdd(&cnt[seg(r, s)], 1u);
        }
    }
    __syncthreads();
    // exclusive scan of the segments' quads; cnt becomes the first quad
    const int per = (nseg + TILE_WG - 1) / TILE_WG, s0 = min(nseg, tid * per), s1 = min(nseg, s0 + per);
    uint32_t tot = 0;
    for (int s = s0; s < s1; ++s) tot += (cnt[s] + 3) / 4;
    scan[tid] = tot;
    __syncthreads();
    for (int off = 1; off < TILE_WG; off <<= 1) {
        const uint32_t a = tid >= off ? scan[tid - off] : 0;
        __syncthreads();
        scan[tid] += a;
        __syncthreads();
    }
    uint32_t at = scan[tid] - tot;
    for (int s = s0; s < s1; ++s) {
        const uint32_t n = (cnt[s] + 3) / 4;
        cnt[s] = at;
        to.sp[b.sp0 + s] = at;
        at += n;
    }
    if (tid == TILE_WG - 1) {
        cnt[nseg] = scan[tid];
        to.sp[b.sp0 + nseg] = scan[tid];
    }
    __syncthreads();
    T *val = (T *)to.val + 4 * b.q0;
    uint16_t *idx = (uint16_t *)(to.idx + b.q0);
    for (int r = wave; r < b.nrows; r += NW) {
        // entries placed so far and first column of every tile, the same in all lanes
        uint32_t fill[TILE_SPLIT], lead[TILE_SPLIT];
#pragma unroll
        for (int k = 0; k < TILE_SPLIT; ++k) fill[k] = lead[k] = 0;
        const int64_t p0 = op.rp[b.row0 + r], p1 = op.rp[b.row0 + r + 1];
        for (int64_t p = p0; p < p1; p += 64) {
            const bool ok = p + lane < p1;
            int loc = 0, s = -1;
            if (ok) s = split((int32_t)(op.ci[p + lane] - b.coff), loc);
            uint32_t rank = 0;
#pragma unroll
            for (int k = 0; k < TILE_SPLIT; ++k) {
                const uint64_t m = __ballot(s == k);
                if (m == 0) continue;
                if (s == k) rank = fill[k] + (uint32_t)__popcll(m & ((1ull << lane) - 1));
                if (fill[k] == 0) lead[k] = (uint32_t)__shfl(loc, __ffsll((unsigned long long)m) - 1);
                fill[k] += (uint32_t)__popcll(m);
            }
            if (ok) {
                const int64_t q = 4 * (int64_t)cnt[seg(r, s)] + rank;
                val[q] = op_vals<T>(op)[p + lane];
                idx[q] = (uint16_t)loc;
            }
        }
        // padding: zero values at the segment's first column
#pragma unroll
        for (int k = 0; k < TILE_SPLIT; ++k) {
            if (k >= b.ntile) break;
            const int g = seg(r, k);
            const uint32_t q = 4 * cnt[g] + fill[k] + lane;
            if (q < 4 * cnt[g + 1]) {
                val[q] = T(0);
                idx[q] = (uint16_t)lead[k];
            }
        }
    }
}

// block lists of the running instances (one workgroup): a scan over the
// instances' block counts, then a wavefront per instance
struct ActLists {
    ActList l[4];  // the tiles' of K, K^T, the other blocks' of K, K^T
};
__global__ __launch_bounds__(TILE_WG) void k_act_lists(Dev d, ActLists lists)
{
    __shared__ int32_t s[TILE_WG], first[TILE_WG], num[TILE_WG];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int o = 0; o < 4; ++o) {
        const ActList &op = lists.l[o];
        if (op.n == 0) continue;
        int32_t carry = 0;
        for (int b0 = 0; b0 < d.batch; b0 += TILE_WG) {
            const int b = b0 + tid;
            const int2 rg = b < d.batch ? op.inst[b] : make_int2(0, 0);
            const int n = b < d.batch && d.st[b].done == 0 ? rg.y - rg.x : 0;
            s[tid] = n;
            first[tid] = rg.x;
            num[tid] = n;
            __syncthreads();
            for (int off = 1; off < TILE_WG; off <<= 1) {
                const int32_t a = tid >= off ? s[tid - off] : 0;
                __syncthreads();
                s[tid] += a;
                __syncthreads();
            }
            for (int k = wave; k < min(TILE_WG, d.batch - b0); k += TILE_WG / 64)
                for (int j = lane; j < num[k]; j += 64)
                    op.act[carry + s[k] - num[k] + j] = op.blk ? op.blk[first[k] + j] : first[k] + j;
            carry += s[TILE_WG - 1];
            __syncthreads();
        }
        if (tid == 0) d.act_cnt[2 + o] = carry;
    }
}

}  // namespace

template <int W, typename T>
static void primal_tile(const Dev &d, const TileOp &op, int j, int avg, Mask mask, hipStream_t s)
{
    const dim3 g(op.grid), wg(W);
    if (mask.p)
        hipLaunchKernelGGL((k_primal_tile<W, T, 0, 1>), g, wg, op.lds, s, d, op, j, mask);
    else if (avg)
        hipLaunchKernelGGL((k_primal_tile<W, T, 1, 0>), g, wg, op.lds, s, d, op, j, mask);
    else
        hipLaunchKernelGGL((k_primal_tile<W, T, 0, 0>), g, wg, op.lds, s, d, op, j, mask);
}

template <int W, typename T>
static void dual_tile(const Dev &d, const TileOp &op, int j, int avg, Mask mask, hipStream_t s)
{
    const dim3 g(op.grid), wg(W);
    if (mask.p)
        hipLaunchKernelGGL((k_dual_tile<W, T, 0, 1>), g, wg, op.lds, s, d, op, j, mask);
    else if (avg)
        hipLaunchKernelGGL((k_dual_tile<W, T, 1, 0>), g, wg, op.lds, s, d, op, j, mask);
    else
        hipLaunchKernelGGL((k_dual_tile<W, T, 0, 0>), g, wg, op.lds, s, d, op, j, mask);
}

template <typename T>
void launch_primal_tile(const Dev &d, const TileOp &op, int j, int avg, Mask mask, hipStream_t s)
{
    if (op.direct)
        primal_tile<256, T>(d, op, j, avg, mask, s);
    else
        primal_tile<1024, T>(d, op, j, avg, mask, s);
}

template <typename T>
void launch_dual_tile(const Dev &d, const TileOp &op, int j, int avg, Mask mask, hipStream_t s)
{
    if (op.direct)
        dual_tile<256, T>(d, op, j, avg, mask, s);
    else
        dual_tile<1024, T>(d, op, j, avg, mask, s);
}

template <typename T>
void launch_tile_build(const OpDev &op, const TileOp &to, hipStream_t s)
{
    hipLaunchKernelGGL(k_tile_build<T>, dim3(to.nblk), dim3(TILE_WG), 0, s, op, to);
}

template <int W, typename T>
static hipError_t tile_attr()
{
    const void *k[6] = {(const void *)k_primal_tile<W, T, 0, 0>, (const void *)k_primal_tile<W, T, 1, 0>,
                        (const void *)k_primal_tile<W, T, 0, 1>, (const void *)k_dual_tile<W, T, 0, 0>,
                        (const void *)k_dual_tile<W, T, 1, 0>,   (const void *)k_dual_tile<W, T, 0, 1>};
    for (const void *f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, TILE_LDS);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T>
hipError_t tile_prepare()
{
    const hipError_t e = tile_attr<256, T>();
    return e == hipSuccess ? tile_attr<1024, T>() : e;
}

void launch_act_lists(const Dev &d, const ActList (&lists)[4], hipStream_t s)
{
    hipLaunchKernelGGL(k_act_lists, dim3(1), dim3(TILE_WG), 0, s, d, ActLists{{lists[0], lists[1], lists[2], lists[3]}});
}

#define TILE_INST(T)                                                                                   \
    template void launch_primal_tile<T>(const Dev &, const TileOp &, int, int, Mask, hipStream_t); \
    template void launch_dual_tile<T>(const Dev &, const TileOp &, int, int, Mask, hipStream_t);   \
    template void launch_tile_build<T>(const OpDev &, const TileOp &, hipStream_t);                     \
    template hipError_t tile_prepare<T>();
TILE_INST(float)
TILE_INST(double)

}  // namespace pdhg
