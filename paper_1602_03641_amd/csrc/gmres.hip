// Kernels of restarted flexible GMRES with classical Gram-Schmidt
// applied twice (CGS2).  The Krylov basis V is stored as (m+1) vectors of
// length ld, one after the other.  Every reduction goes through per-block
// partials summed in a fixed order (deterministic); the Hessenberg column is
// reduced on the device and read by the host once per iteration.
#include "reduce.h"
#include "sell.h"

namespace vag {

namespace {

constexpr int kT = 256;
// Most basis vectors whose entries a thread holds at once.  The reductions' grid
// is 512 blocks of 256 threads (2 wavefronts per SIMD), so what is read ahead
// has to come from the loads of one thread: all basis entries of its row, in up
// to 64 VGPRs, before the first is used.
constexpr int kBasis = 32;

#define GS(i, n) \
    for (int64_t i = (int64_t)xcd_block() * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// y = A x; SPLIT: four lanes per row
template <bool SPLIT, class V, class T>
__global__ __launch_bounds__(kT) void gm_spmv_kernel(Sell<V> A, const T *__restrict__ x, T *__restrict__ y) {
    const auto f = [&](int32_t j) { return (double)x[j]; };
    if constexpr (SPLIT) {
        const int32_t i = split_row<kT, true>();
        const double t = lane_row(A, i, f).template sum<double, 1>([](double v) { return v; });
        if ((threadIdx.x & 63) < kSplitRows && i < A.n) y[i] = (T)t;
    } else {
        GS(i, A.n) y[i] = (T)sell_row_apply<V, double>(A, (int32_t)i, f);
    }
}

// v[i] = entry r of basis vector i, i < k
template <int K, class T>
__device__ inline void basis_row(const T *__restrict__ V, int64_t ld, int64_t r, int k, T (&v)[K]) {
#pragma unroll
    for (int i = 0; i < K; ++i)
        if (i < k) v[i] = V[(int64_t)i * ld + r];
}

// parts[(c*K + i) * G + bx] = partial of <V_{c*K+i}, w> over block bx
template <int K, class T>
__device__ inline void dot_partials(double (&v)[K], int c0, int k, double *parts) {
    block_reduce<OpSum, K, kT>(v);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (c0 + i < k) parts[(size_t)(c0 + i) * gridDim.x + blockIdx.x] = v[i];
    }
}
template <int K, class T>
__global__ __launch_bounds__(kT) void gm_multidot_kernel(int32_t n, int k, const T *__restrict__ V, int64_t ld,
                                                         const T *__restrict__ w, double *__restrict__ parts) {
    const int c0 = blockIdx.y * K;
    double v[K];
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = 0.0;
    GS(r, n) {
        T b[K];
        basis_row<K>(V + (int64_t)c0 * ld, ld, r, k - c0, b);
        const double wr = (double)w[r];
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (c0 + i < k) v[i] += (double)b[i] * wr;
    }
    dot_partials<K, T>(v, c0, k, parts);
}

// h[i] = sum of the G partials of dot i (one block per dot)
__global__ __launch_bounds__(kT) void gm_hreduce_kernel(const double *__restrict__ parts, int G,
                                                        double *__restrict__ h) {
    const double t = sum_parts<OpSum, kT>(parts + (size_t)blockIdx.x * G, G);
    if (threadIdx.x == 0) h[blockIdx.x] = t;
}

// w -= sum_{i<k} h[i] V_i; NORM: and partials of ||w||^2
template <int K, bool NORM, class T>
__global__ __launch_bounds__(kT) void gm_multiaxpy_kernel(int32_t n, int k, const T *__restrict__ V, int64_t ld,
                                                          const double *__restrict__ h, T *__restrict__ w,
                                                          double *__restrict__ parts) {
    double v[1] = {0.0};
    GS(r, n) {
        double t = (double)w[r];
        for (int c0 = 0; c0 < k; c0 += K) {
            T b[K];
            basis_row<K>(V + (int64_t)c0 * ld, ld, r, k - c0, b);
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (c0 + i < k) t -= h[c0 + i] * (double)b[i];
        }
        const T tw = (T)t;
        w[r] = tw;
        if (NORM) v[0] += (double)tw * (double)tw;
    }
    if constexpr (NORM) block_partials<OpSum, 1, kT>(v, parts, gridDim.x);
}

// The first subtraction and the second pass's dots while the basis row is at
// hand (k <= K): w -= sum h[i] V_i, parts as in gm_multidot_kernel of the new w.
// A step of the orthogonalisation reads the basis three times instead of four:
// 2.1 M rows, 1 to 26 vectors, mean of a step 325 -> 157 us.
template <int K, class T>
__global__ __launch_bounds__(kT) void gm_axpy_dots_kernel(int32_t n, int k, const T *__restrict__ V, int64_t ld,
                                                          const double *__restrict__ h, T *__restrict__ w,
                                                          double *__restrict__ parts) {
    double v[K];
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = 0.0;
    GS(r, n) {
        T b[K];
        basis_row<K>(V, ld, r, k, b);
        double t = (double)w[r];
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i < k) t -= h[i] * (double)b[i];
        const T tw = (T)t;
        w[r] = tw;
        const double wr = (double)tw;
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i < k) v[i] += (double)b[i] * wr;
    }
    dot_partials<K, T>(v, 0, k, parts);
}

// out = s * (the vector w), s = 1 / sqrt(sum of the partials); hn = sqrt(...)
template <class T>
__global__ __launch_bounds__(kT) void gm_normalize_kernel(int32_t n, const double *__restrict__ parts, int G,
                                                          const T *__restrict__ w, T *__restrict__ out,
                                                          double *__restrict__ hn) {
    const double nrm = sqrt(sum_parts<OpSum, kT>(parts, G));
    if (blockIdx.x == 0 && threadIdx.x == 0) *hn = nrm;
    const double s = nrm > 0.0 ? 1.0 / nrm : 0.0;
    GS(r, n) out[r] = (T)(s * (double)w[r]);
}

// x += sum_{i<k} y[i] V_i, the sum rounded to T first
template <int K, class T>
__global__ __launch_bounds__(kT) void gm_combine_kernel(int32_t n, int k, const T *__restrict__ V, int64_t ld,
                                                        const double *__restrict__ y, T *__restrict__ x) {
    GS(r, n) {
        double s = 0.0;
        for (int c0 = 0; c0 < k; c0 += K) {
            T b[K];
            basis_row<K>(V + (int64_t)c0 * ld, ld, r, k - c0, b);
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (c0 + i < k) s += y[c0 + i] * (double)b[i];
        }
        x[r] = (T)((double)x[r] + (double)(T)s);
    }
}

// r = b - A x, partials of ||r||^2
template <class V, class T>
__global__ __launch_bounds__(kT) void gm_residual_kernel(Sell<V> A, const T *__restrict__ b, const T *__restrict__ x,
                                                         T *__restrict__ r, double *__restrict__ parts) {
    double v[1] = {0.0};
    GS(i, A.n) {
        const double t =
            (double)b[i] - sell_row_apply<V, double>(A, (int32_t)i, [&](int32_t j) { return (double)x[j]; });
        const T tr = (T)t;
        r[i] = tr;
        v[0] += (double)tr * (double)tr;
    }
    block_partials<OpSum, 1, kT>(v, parts, gridDim.x);
}

}  // namespace

int gmres_grid(int64_t n) { return (int)reduce_grid(n, kT); }

template <class V, class T>
void launch_gm_spmv(hipStream_t s, Sell<V> A, const T *x, T *y) {
    if (A.n <= 0) return;
    // no partials, so no limit on the blocks: 2.1 M rows 162 -> 126 us
    if (krylov_shape(A.n).split)
        hipLaunchKernelGGL((gm_spmv_kernel<true, V, T>), dim3((A.n + kT / kChains - 1) / (kT / kChains)), dim3(kT), 0,
                           s, A, x, y);
    else
        hipLaunchKernelGGL((gm_spmv_kernel<false, V, T>), dim3(((int64_t)A.n + kT - 1) / kT), dim3(kT), 0, s, A, x, y);
    VAG_HIP(hipGetLastError());
}

// call with K: the smallest of 8, 16 and kBasis that holds k vectors (else
// kBasis at a time)
#define GM_BASIS(k, call)                    \
    do {                                     \
        if ((k) <= 8) {                      \
            constexpr int K = 8;             \
            call;                            \
        } else if ((k) <= 16) {              \
            constexpr int K = 16;            \
            call;                            \
        } else {                             \
            constexpr int K = kBasis;        \
            call;                            \
        }                                    \
        VAG_HIP(hipGetLastError());          \
    } while (0)

template <class T>
void launch_gm_orthogonalize(hipStream_t s, int32_t n, int k, const T *V, int64_t ld, T *w, double *parts,
                             double *h1, double *h2, double *nparts) {
    const int G = gmres_grid(n);
    const auto dots = [&] {
        GM_BASIS(k, hipLaunchKernelGGL((gm_multidot_kernel<K, T>), dim3(G, (k + K - 1) / K), dim3(kT), 0, s, n, k, V,
                                       ld, w, parts));
    };
    const auto sums = [&](double *h) {
        hipLaunchKernelGGL(gm_hreduce_kernel, dim3(k), dim3(kT), 0, s, parts, G, h);
        VAG_HIP(hipGetLastError());
    };
    dots();
    sums(h1);
    if (k <= kBasis) {
        GM_BASIS(k, hipLaunchKernelGGL((gm_axpy_dots_kernel<K, T>), dim3(G), dim3(kT), 0, s, n, k, V, ld, h1, w,
                                       parts));
    } else {
        GM_BASIS(k, hipLaunchKernelGGL((gm_multiaxpy_kernel<K, false, T>), dim3(G), dim3(kT), 0, s, n, k, V, ld, h1, w,
                                       nparts));
        dots();
    }
    sums(h2);
    GM_BASIS(k, hipLaunchKernelGGL((gm_multiaxpy_kernel<K, true, T>), dim3(G), dim3(kT), 0, s, n, k, V, ld, h2, w,
                                   nparts));
}

template <class T>
void launch_gm_normalize(hipStream_t s, int32_t n, const double *nparts, const T *w, T *out, double *hn) {
    const int G = gmres_grid(n);
    hipLaunchKernelGGL((gm_normalize_kernel<T>), dim3(G), dim3(kT), 0, s, n, nparts, G, w, out, hn);
    VAG_HIP(hipGetLastError());
}

template <class T>
void launch_gm_combine(hipStream_t s, int32_t n, int k, const T *V, int64_t ld, const double *y, T *x) {
    GM_BASIS(k, hipLaunchKernelGGL((gm_combine_kernel<K, T>), dim3(gmres_grid(n)), dim3(kT), 0, s, n, k, V, ld, y, x));
}

template <class V, class T>
void launch_gm_residual(hipStream_t s, Sell<V> A, const T *b, const T *x, T *r, double *nparts) {
    hipLaunchKernelGGL((gm_residual_kernel<V, T>), dim3(gmres_grid(A.n)), dim3(kT), 0, s, A, b, x, r, nparts);
    VAG_HIP(hipGetLastError());
}

#define GM_INST(T)                                                                                               \
    template void launch_gm_spmv<T, T>(hipStream_t, Sell<T>, const T *, T *);                                    \
    template void launch_gm_orthogonalize<T>(hipStream_t, int32_t, int, const T *, int64_t, T *, double *,      \
                                             double *, double *, double *);                                     \
    template void launch_gm_normalize<T>(hipStream_t, int32_t, const double *, const T *, T *, double *);        \
    template void launch_gm_combine<T>(hipStream_t, int32_t, int, const T *, int64_t, const double *, T *);      \
    template void launch_gm_residual<T, T>(hipStream_t, Sell<T>, const T *, const T *, T *, double *);
GM_INST(double)
GM_INST(float)

}  // namespace vag
