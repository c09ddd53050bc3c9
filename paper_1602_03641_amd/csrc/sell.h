// Row kernels on sliced ELL (64-row slices, column-major inside a slice).
#pragma once

#include <utility>

#include "reduce.h"

namespace vag {

// sum over the levels k of the slice of A[row, k] * f(col(k)), kChains
// independent accumulation chains (chain c takes the levels k = c mod
// kChains) so that several gathers are in flight per lane.  The summation
// order is fixed.  The level index k, the slice's start b0 and its width w are
// the same for every lane (the wavefront holds the slice's 64 rows), so the
// loop control and the per-level column bases stay in scalar registers.
constexpr int kChains = 4;
template <bool NT, class V, class Acc, class F, class Col>
__device__ inline void sell_row_chains(const Sell<V> &A, int64_t b0, int32_t w, int lane, Acc *s, F f, Col col) {
    int32_t k = 0;
    for (; k + kChains <= w; k += kChains) {
#pragma unroll
        for (int c = 0; c < kChains; ++c) {
            const int64_t p = b0 + 64 * (int64_t)(k + c) + lane;
            s[c] += (Acc)ld_matrix<NT>(&A.val[p]) * f(col(p, k + c));
        }
    }
#pragma unroll
    for (int c = 0; c < kChains - 1; ++c)
        if (k + c < w) {
            const int64_t p = b0 + 64 * (int64_t)(k + c) + lane;
            s[c] += (Acc)ld_matrix<NT>(&A.val[p]) * f(col(p, k + c));
        }
}

// Row `row` of A applied to f.  Every caller runs one thread per row in blocks
// of whole wavefronts, so the active lanes of a wavefront are rows of one
// slice and lane = row mod 64.
template <class V, class Acc, class F>
__device__ inline Acc sell_row_apply(const Sell<V> &A, int32_t row, F f) {
    const int32_t sl = __builtin_amdgcn_readfirstlane(row >> 6);
    const int64_t b0 = A.ptr[sl], b1 = A.ptr[sl + 1];
    const int32_t w = (int32_t)((b1 - b0) >> 6);
    const int lane = row & 63;
    Acc s[kChains];
#pragma unroll
    for (int c = 0; c < kChains; ++c) s[c] = 0;
    // 16-bit columns where the slice's first level has a base: level k's base
    // is cbase[b0 / 64 + k]
    const int32_t *cb = A.col16 && w > 0 && A.cbase[b0 >> 6] >= 0 ? A.cbase + (b0 >> 6) : nullptr;
    if (cb) {
        if (A.nt)
            sell_row_chains<true, V, Acc>(A, b0, w, lane, s, f, [&](int64_t p, int32_t k) {
                return cb[k] + (int32_t)ld_matrix<true>(&A.col16[p]);
            });
        else
            sell_row_chains<false, V, Acc>(A, b0, w, lane, s, f,
                                           [&](int64_t p, int32_t k) { return cb[k] + (int32_t)A.col16[p]; });
    } else {
        if (A.nt)
            sell_row_chains<true, V, Acc>(A, b0, w, lane, s, f,
                                          [&](int64_t p, int32_t) { return ld_matrix<true>(&A.col[p]); });
        else
            sell_row_chains<false, V, Acc>(A, b0, w, lane, s, f, [&](int64_t p, int32_t) { return A.col[p]; });
    }
#pragma unroll
    for (int w2 = kChains / 2; w2 > 0; w2 >>= 1)
#pragma unroll
        for (int c = 0; c < w2; ++c) s[c] += s[c + w2];
    if (A.dg) s[0] += (Acc)A.dg[row] * f(row);
    return s[0];
}

// A row with kChains lanes, for matrices too small to fill the device with one
// lane per row: a wavefront holds 64 / kChains consecutive rows, lane group g
// taking the entries g, g + kChains, ... in turn.  load() reads a lane's
// columns and values of a batch (a row of up to 32 entries), then what
// gather(j) returns for each column, so that the row waits for one chain of
// loads, and that while the kernel forms the scalars it needs; sum() then
// combines each value with use(gathered).  A lane past the row's end repeats
// its first entry and adds nothing.  Called by whole wavefronts.
constexpr int kSplitRows = 64 / kChains;  // rows per wavefront
template <class V, class Gather>
struct LaneRow {
    static constexpr int B = 8;
    using Raw = decltype(std::declval<Gather>()(0));
    const Sell<V> &A;
    const int32_t row;
    Gather gather;
    int64_t q, b1;
    V v[B];
    Raw x[B];
    __device__ inline LaneRow(const Sell<V> &A_, int32_t row_, Gather g) : A(A_), row(row_), gather(g) {
        const bool in = row < A.n;
        const int32_t r = in ? row : 0;
        b1 = A.ptr[(r >> 6) + 1];
        q = A.ptr[r >> 6] + (r & 63) + (int64_t)((threadIdx.x & 63) / kSplitRows) * 64;
        if (!in) b1 = q;  // no entries
        load();
    }
    __device__ inline void load() {
        if (q >= b1) return;
        int32_t c[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int64_t p = q + b * kChains * 64;
            c[b] = A.col[p < b1 ? p : q];
            v[b] = A.val[p < b1 ? p : q];
        }
#pragma unroll
        for (int b = 0; b < B; ++b) x[b] = gather(c[b]);
    }
    // ACC accumulators a lane: 1, the chains of sell_row_apply, combined in its
    // order (the same bits); 2, the order of the V-cycle kernels on small
    // levels.  Valid in the wavefront's first kSplitRows lanes.
    template <class Acc, int ACC, class Use>
    __device__ inline Acc sum(Use use) {
        Acc s[ACC];
#pragma unroll
        for (int k = 0; k < ACC; ++k) s[k] = 0;
        while (q < b1) {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const Acc t = s[b % ACC] + (Acc)v[b] * use(x[b]);
                s[b % ACC] = q + b * kChains * 64 < b1 ? t : s[b % ACC];
            }
            q += B * kChains * 64;
            load();
        }
        Acc t = s[0];
        if constexpr (ACC == 2) {
            t += s[1];
            t += down<16>(t);
            t += down<32>(t);
        } else {
            t += down<32>(t);
            t += down<16>(t);
        }
        if (A.dg && row < A.n) t += (Acc)A.dg[row] * use(gather(row));
        return t;
    }
    template <int O>
    __device__ static inline double down(double t) {
        return lane_down<O>(t);
    }
    template <int O>
    __device__ static inline float down(float t) {
        return __int_as_float(lane_down<O>(__float_as_int(t)));
    }
};
template <class V, class Gather>
__device__ inline LaneRow<V, Gather> lane_row(const Sell<V> &A, int32_t row, Gather g) {
    return LaneRow<V, Gather>(A, row, g);
}

// The rows of a Krylov kernel of NT threads, one lane per row: row(i, (A f)_i,
// v) adds the row's share of NV reductions to v, whose partials go to p(k).
// slices: one pass (the grid covers the partials' rows); else a grid-stride
// loop.  XCD: blocks numbered by xcd_block(); the partials are then those of a
// launch over 1024-row blocks so numbered.
template <bool XCD>
__device__ inline int slice_place(int slice, int G) {
    return XCD ? (int)(xcd_unblock((unsigned)slice >> 4, (unsigned)G >> 4) * 16 + (slice & 15)) : slice;
}
template <int NT, int NV, bool XCD, class V, class Acc, class F, class Row, class P>
__device__ inline void krylov_rows(const Sell<V> &A, bool slices, int G, F f, Row row, P p) {
    const int64_t blk = XCD ? xcd_block() : blockIdx.x;
    double v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = 0.0;
    for (int64_t i = blk * NT + threadIdx.x; i < A.n; i += (int64_t)gridDim.x * NT)
        row((int32_t)i, sell_row_apply<V, Acc>(A, (int32_t)i, f), v);
    krylov_put<NT, NV>(slices, p, slice_place<XCD>((int)((blk * NT + threadIdx.x) >> 6), G), v);
}
// The same with kChains lanes per row and slices: the kernel has read its row
// into r (lane_row of split_row) and gives the sum s to row.
template <int NT, bool XCD>
__device__ inline int32_t split_row() {
    const int64_t blk = XCD ? xcd_block() : blockIdx.x;
    return (int32_t)(blk * (NT / kChains) + (threadIdx.x >> 6) * kSplitRows + (threadIdx.x & 63) % kSplitRows);
}
template <int NT, int NV, bool XCD, bool PLACE = XCD, class Acc, class Row, class P>
__device__ inline void split_rows(int32_t n, int G, int32_t i, Acc s, Row row, P p) {
    __shared__ double share[NV][NT / kChains];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = 0.0;
    if (lane < kSplitRows) {
        if (i < n) row(i, s, v);
#pragma unroll
        for (int k = 0; k < NV; ++k) share[k][wave * kSplitRows + lane] = v[k];
    }
    __syncthreads();
    if (wave < NT / kChains / 64) {  // whole wavefronts: one slice each
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = share[k][threadIdx.x];
        const int64_t blk = XCD ? xcd_block() : blockIdx.x;
        krylov_put<NT, NV>(true, p, slice_place<PLACE>((int)(blk * (NT / kChains / 64) + wave), G), v);
    }
}

// Evaluates call (a launch of some kern<SPLIT, ...> over matrix rows, blocks of
// `threads`) in the given shape
#define VAG_ROWS_LAUNCH(shape, call)            \
    do {                                        \
        const KrylovShape ks = shape;           \
        if (ks.split) {                         \
            constexpr bool SPLIT = true;        \
            constexpr int threads = kSplitThreads; \
            call;                               \
        } else {                                \
            constexpr bool SPLIT = false;       \
            constexpr int threads = kKrylovThreads; \
            call;                               \
        }                                       \
        VAG_HIP(hipGetLastError());             \
    } while (0)

// The slots of row i of a sliced-ELL array, kSlots at a time: load(j, q) for
// the batch (a slot past the row repeats its first, whose lines are there
// already), so that a row waits for one chain of loads a batch and not one a
// slot, then use(j, q) in slot order for those that exist.
constexpr int kSlots = 8;
template <class Load, class Use>
__device__ inline void row_slots(const int64_t *__restrict__ ptr, int64_t i, Load load, Use use) {
    const int64_t b1 = ptr[(i >> 6) + 1];
    for (int64_t q0 = ptr[i >> 6] + (i & 63); q0 < b1; q0 += 64 * kSlots) {
#pragma unroll
        for (int j = 0; j < kSlots; ++j) load(j, q0 + 64 * j < b1 ? q0 + 64 * j : q0);
#pragma unroll
        for (int j = 0; j < kSlots; ++j)
            if (q0 + 64 * j < b1) use(j, q0 + 64 * j);
    }
}

}  // namespace vag
