// Deterministic reductions for wave64 devices without grid-wide fences.
//
// A reducing kernel writes one partial per block (block_partials).  The total
// is formed later, after a kernel boundary has made the partials visible: either
// redundantly by every block of the consuming kernel (sum_parts, all blocks
// read the same partials in the same order and get the same bits), or by a
// one-block finishing kernel.  The summation order depends only on the launch
// shape, never on timing, so results are bitwise reproducible.
#pragma once

#include "vag_internal.h"

namespace vag {

// The workgroups of a launch are dealt to the 8 XCDs in turn (block b to XCD
// b mod 8), each XCD with its own L2.  xcd_block() renumbers the blocks so
// that every XCD receives one contiguous run of block indices: neighbouring
// rows then share an L2, and the gathers of a row's neighbours (and of an
// aggregate's members) hit lines that the same XCD has already fetched.  A
// bijection of [0, gridDim.x).
__device__ inline unsigned xcd_block() {
    const unsigned nb = gridDim.x, b = blockIdx.x, q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}

struct OpSum {
    __device__ static double id() { return 0.0; }
    __device__ static double op(double a, double b) { return a + b; }
};
struct OpMin {
    __device__ static double id() { return __builtin_inf(); }
    __device__ static double op(double a, double b) { return a < b ? a : b; }
};

// The value of lane i + O for the lanes a reduction tree asks for it (O = 32:
// i < 32; O = 16: even rows of 16 lanes; O = 8, 4, 2, 1: inside a row of 16, 0
// past its end), by lane swaps and row shifts of the vector unit: a shuffle
// through LDS takes about three times as long.
template <int O>
__device__ inline int lane_down(int v) {
    if constexpr (O == 32) return (int)__builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
    else if constexpr (O == 16) return (int)__builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
    else return __builtin_amdgcn_update_dpp(0, v, 0x100 | O, 0xf, 0xf, true);  // row_shl
}
template <int O>
__device__ inline double lane_down(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)lane_down<O>((int)(uint32_t)u), hi = (uint32_t)lane_down<O>((int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
template <class Op>
__device__ inline double wave_reduce(double v) {
    v = Op::op(v, lane_down<32>(v));
    v = Op::op(v, lane_down<16>(v));
    v = Op::op(v, lane_down<8>(v));
    v = Op::op(v, lane_down<4>(v));
    v = Op::op(v, lane_down<2>(v));
    v = Op::op(v, lane_down<1>(v));
    return v;  // valid in lane 0
}

// Reduces NV values per thread over the block; results valid in every thread.
template <class Op, int NV, int NT>
__device__ inline void block_reduce(double (&v)[NV]) {
    __shared__ double lds[NV][NT / 64];
    __shared__ double res[NV];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double t = wave_reduce<Op>(v[k]);
        if (lane == 0) lds[k][w] = t;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double t = lds[threadIdx.x][0];
        for (int i = 1; i < NT / 64; ++i) t = Op::op(t, lds[threadIdx.x][i]);
        res[threadIdx.x] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = res[k];
    __syncthreads();
}

// Writes the block's reduction of NV values to parts[k * stride + blockIdx.x].
template <class Op, int NV, int NT>
__device__ inline void block_partials(double (&v)[NV], double *parts, int stride) {
    block_reduce<Op, NV, NT>(v);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) parts[(size_t)k * stride + blockIdx.x] = v[k];
    }
}

// Total of nparts partials, identical in every thread of every block.
template <class Op, int NT>
__device__ inline double sum_parts(const double *parts, int nparts) {
    double v[1] = {Op::id()};
    for (int i = threadIdx.x; i < nparts; i += NT) v[0] = Op::op(v[0], parts[i]);
    block_reduce<Op, 1, NT>(v);
    return v[0];
}

// Totals of NV arrays of nparts partials (p(k) names the k-th): one pass, one
// block reduction.
template <class Op, int NT, int NV, class P>
__device__ inline void sum_parts_of(P p, int nparts, double (&v)[NV]) {
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = Op::id();
    for (int i = threadIdx.x; i < nparts; i += NT)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = Op::op(v[k], p(k)[i]);
    block_reduce<Op, NV, NT>(v);
}

// The place of logical block b of xcd_block()'s numbering: the inverse map.
__device__ inline unsigned xcd_unblock(unsigned b, unsigned nb) {
    const unsigned q = nb >> 3, r = nb & 7, big = r * (q + 1);
    const unsigned x = b < big ? b / (q + 1) : r + (b - big) / max(q, 1u);
    return (b - (x * q + (x < r ? x : r))) * 8 + x;
}

// Totals of NV arrays of G slice sums (see KrylovShape), in every thread: the
// 16 slices of 1024 rows one after the other, then the shuffle tree and the
// wavefront totals as block_reduce and sum_parts combine blocks of 1024 rows.
static_assert(kSplitMaxRows <= kSplitMaxBcg, "the most slices that slice_sums adds up");
template <int NT, int NV, class P>
__device__ inline void slice_sums(P p, int G, double (&v)[NV]) {
    __shared__ double lds[NV][(kSplitMaxBcg / kSliceRows + 1023) / 1024];
    const int lane = threadIdx.x & 63, nc = (G + 1023) / 1024;
    for (int c = threadIdx.x >> 6; c < nc; c += NT / 64) {
        const int at = (c * 64 + lane) * 16;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double t = 0.0;
            if (at < G) {
                const double2 *q = reinterpret_cast<const double2 *>(p(k) + at);
                double2 w[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = q[j];
                t = w[0].x + w[0].y;
#pragma unroll
                for (int j = 1; j < 8; ++j) {
                    t += w[j].x;
                    t += w[j].y;
                }
            }
            t = wave_reduce<OpSum>(t);
            if (lane == 0) lds[k][c] = t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = lds[k][0];
        for (int c = 1; c < nc; ++c) v[k] += lds[k][c];
    }
    __syncthreads();
}

// Totals of NV Krylov reductions, either form of their partials
template <int NT, int NV, class P>
__device__ inline void krylov_sums(bool slices, P p, int G, double (&v)[NV]) {
    if (slices)
        slice_sums<NT>(p, G, v);
    else
        sum_parts_of<OpSum, NT>(p, G, v);
}

// A thread's share v[k] of NV reductions as partials in p(k): the sum of the
// wavefront's 64 consecutive rows as slice `slice`, or the block's sum (null:
// not wanted).
template <int NT, int NV, class P>
__device__ inline void krylov_put(bool slices, P p, int slice, double (&v)[NV]) {
    if (slices) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const double t = wave_reduce<OpSum>(v[k]);
            if ((threadIdx.x & 63) == 0 && p(k)) p(k)[slice] = t;
        }
    } else {
        block_reduce<OpSum, NV, NT>(v);
        if (threadIdx.x == 0)
#pragma unroll
            for (int k = 0; k < NV; ++k)
                if (p(k)) p(k)[blockIdx.x] = v[k];
    }
}

// A value for the host, which polls pinned memory (or reads it after the next
// synchronisation): no copy to queue and wait for.
__device__ inline void host_put(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

// Ends a Krylov solve (one thread calls it): the later kernels return at
// once, and the host, which looks at its flag before it queues an iteration,
// queues no more of them.
__device__ inline void krylov_done(PcgState *st, int converged, double rr) {
    st->done = 1;
    st->converged = converged;
    st->rr = rr;
    if (st->host_done) host_put(st->host_done, 1);
}

inline unsigned reduce_grid(int64_t n_items, int threads) {
    int64_t b = (n_items + threads - 1) / threads;
    if (b > kReduceBlocks) b = kReduceBlocks;
    if (b < 1) b = 1;
    return (unsigned)b;
}

// one-block kernel: out[k] = Op-total of parts[k*stride .. k*stride+nparts)
void launch_finalize_sum(hipStream_t s, const double *parts, int stride, int nparts, int nv, double *out);
void launch_finalize_min(hipStream_t s, const double *parts, int stride, int nparts, int nv, double *out);

}  // namespace vag
