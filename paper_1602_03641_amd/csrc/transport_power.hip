// Several explicit steps per launch: the step is linear (c^{n+1} = T c^n, see
// transport.hip), so on a small mesh, where a step is one launch that lasts
// 3.6 us whatever it computes, calls of many steps apply T^4 (or T^2) instead.
// Rows hold their entries side by side in a fixed width W (col and val at
// row * W, len[row] of them); row nrow is the constant control volume.  A row
// that needs more than W entries sets *over: the power is then not used.
// All entries of T are nonnegative and its rows sum to at most one, so the
// products add no cancellation to what the steps have.
#include "reduce.h"

namespace vag {

namespace {

constexpr int kHash = 256;      // table of a product's row
constexpr int kStepLanes = 16;  // per row of a step

}  // namespace

// T with its diagonal, one wavefront per slice of the operator
__global__ __launch_bounds__(kSliceRows) void power_base_kernel(UpwindOp T, PowerRows R, int *over) {
    const int32_t sl = blockIdx.x;
    const int lane = threadIdx.x;
    const uint16_t m = T.meta[sl * kSliceRows + lane];
    const int32_t i = sl * kSliceRows + (m >> 8);
    const bool row = i < T.nrow;
    const int cnt = row ? (m & 255) : 0;
    const int width = __shfl(cnt, 0, 64);  // the slice's rows are sorted longest first
    const int64_t o = (int64_t)i * R.W;
    bool fits = cnt + 1 <= R.W;
    int64_t p = T.slice_ptr[sl] + lane;
    for (int k = 0; k < width; ++k) {
        const bool has = cnt > k;
        const int n = __popcll(__ballot(has));
        if (has && fits) {
            R.col[o + k] = T.tcol[p];
            R.val[o + k] = T.tval[p];
        }
        p += n;
    }
    if (row && fits) {
        R.col[o + cnt] = i;
        R.val[o + cnt] = T.tdiag[i];
        R.len[i] = cnt + 1;
    }
    if (!fits) {
        if (row) R.len[i] = 0;
        *over = 1;
    }
    if (sl == 0 && lane == 0) {
        const int64_t c = (int64_t)T.nrow * R.W;
        R.col[c] = T.nrow;
        R.val[c] = 1.0;
        R.len[T.nrow] = 1;
    }
}

// C = A A, one wavefront per row: the rows that row i of A names, in its order,
// their entries by the lanes, summed in a table in LDS and stored in column
// order.  Deterministic: a row's columns differ, so no two lanes add to one
// entry at a time.
__global__ __launch_bounds__(256) void power_square_kernel(int32_t n, PowerRows A, PowerRows C, int *over) {
    __shared__ int32_t key[4][kHash], list[4][kHash];
    __shared__ double sum[4][kHash];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int32_t i = (int32_t)blockIdx.x * 4 + wave;
    if (i >= n) return;  // whole wavefronts, and no barriers below
    int32_t *K = key[wave], *L = list[wave];
    double *S = sum[wave];
    for (int k = lane; k < kHash; k += 64) {
        K[k] = -1;
        S[k] = 0.0;
    }
    const int len = A.len[i];
    const int32_t cl = lane < len ? A.col[(int64_t)i * A.W + lane] : 0;
    const double vl = lane < len ? A.val[(int64_t)i * A.W + lane] : 0.0;
    const int nl = lane < len ? A.len[cl] : 0;
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    fence();
    bool full = len > 64 || A.W > 64;
    for (int k0 = 0; k0 < len && !full; k0 += 4) {  // four rows' loads in flight
        int32_t c[4];
        double v[4], a[4];
        bool on[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = min(k0 + u, len - 1);
            const int32_t r = __shfl(cl, k, 64);
            a[u] = __shfl(vl, k, 64);
            on[u] = k0 + u < len && lane < __shfl(nl, k, 64);
            const int64_t q = (int64_t)r * A.W + (on[u] ? lane : 0);
            c[u] = A.col[q];
            v[u] = A.val[q];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bool placed = !on[u];
            uint32_t h = ((uint32_t)c[u] * 2654435761u) >> 24;
            for (int probe = 0; probe < kHash && !placed; ++probe) {
                const int32_t prev = atomicCAS(&K[h], -1, c[u]);
                if (prev == -1 || prev == c[u]) {
                    S[h] = fma(a[u], v[u], S[h]);
                    placed = true;
                } else {
                    h = (h + 1) & (kHash - 1);
                }
            }
            if (__ballot(!placed)) full = true;
            fence();
        }
    }
    int nd = 0;
    for (int k0 = 0; k0 < kHash; k0 += 64) {
        const bool used = K[k0 + lane] >= 0;
        const uint64_t mask = __ballot(used);
        if (used) L[nd + __popcll(mask & ((1ull << lane) - 1))] = k0 + lane;
        nd += __popcll(mask);
    }
    fence();
    if (full || nd > C.W) {
        if (lane == 0) {
            C.len[i] = 0;
            *over = 1;
        }
        return;
    }
    for (int e = lane; e < nd; e += 64) {
        const int32_t c = K[L[e]];
        int rank = 0;
        for (int u = 0; u < nd; ++u) rank += K[L[u]] < c;
        C.col[(int64_t)i * C.W + rank] = c;
        C.val[(int64_t)i * C.W + rank] = S[L[e]];
    }
    if (lane == 0) C.len[i] = nd;
}

// c_out = R c_in, kStepLanes lanes per row, their sums by a fixed tree
__global__ __launch_bounds__(256) void power_step_kernel(int32_t n, PowerRows R, const double *__restrict__ c_in,
                                                         double *__restrict__ c_out) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kStepLanes;
    const int q = threadIdx.x % kStepLanes;
    const int len = i < n ? R.len[i] : 0;
    const int64_t o = (i < n ? i : 0) * R.W;
    double t = 0.0;
    for (int k0 = q; k0 < len; k0 += 4 * kStepLanes) {  // four entries' loads in flight
        int32_t c[4];
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * kStepLanes;
            c[u] = R.col[o + (k < len ? k : q)];
            v[u] = R.val[o + (k < len ? k : q)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double x = c_in[c[u]];
            t += k0 + u * kStepLanes < len ? v[u] * x : 0.0;
        }
    }
#pragma unroll
    for (int d = kStepLanes / 2; d > 0; d >>= 1) t += __shfl_down(t, d, kStepLanes);
    if (q == 0 && i < n) c_out[i] = t;
}

void launch_power_base(hipStream_t s, const UpwindOp &T, const PowerRows &R, int *over) {
    hipLaunchKernelGGL(power_base_kernel, dim3((T.nrow + kSliceRows - 1) / kSliceRows), dim3(kSliceRows), 0, s, T, R,
                       over);
    VAG_HIP(hipGetLastError());
}
void launch_power_square(hipStream_t s, int32_t n, const PowerRows &A, const PowerRows &C, int *over) {
    hipLaunchKernelGGL(power_square_kernel, dim3((n + 3) / 4), dim3(256), 0, s, n, A, C, over);
    VAG_HIP(hipGetLastError());
}
void launch_power_step(hipStream_t s, int32_t n, const PowerRows &R, const double *c_in, double *c_out) {
    hipLaunchKernelGGL(power_step_kernel, dim3((unsigned)(((int64_t)n * kStepLanes + 255) / 256)), dim3(256), 0, s, n, R,
                       c_in, c_out);
    VAG_HIP(hipGetLastError());
}

}  // namespace vag
