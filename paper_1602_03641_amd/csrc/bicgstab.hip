// Kernels of right-preconditioned BiCGStab (van der Vorst's stabilised
// bi-conjugate gradients, the alternative Krylov method of the paper's solver
// study, §5.3) with every scalar kept on the device: each kernel forms the
// scalars it needs from the per-block partials of the previous kernels
// (summed in a fixed order by every block, so the result is bitwise
// reproducible), and the host only queues iterations and reads the state
// every few iterations, as for CG.
//
// Iteration k (rhat = r_0 fixed; p, v, s, t as in the method):
//   rho_k   = rhat . r_k
//   beta    = (rho_k / rho_{k-1}) (alpha_{k-1} / omega_{k-1})
//   p       = r + beta (p - omega_{k-1} v)          (p = r at the start)
//   phat    = M^-1 p,   v = A phat,   alpha_k = rho_k / (rhat . v)
//   s       = r - alpha_k v                           (done if |s| is small)
//   shat    = M^-1 s,   t = A shat,   omega_k = (t . s) / (t . t)
//   x      += alpha_k phat + omega_k shat,   r = s - omega_k t
#include "reduce.h"
#include "sell.h"

namespace vag {

namespace {

constexpr int kT = kKrylovThreads;

#define GSB(i, n) \
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// partial slots: rho(k) parity 0/1, rhat.v, t.s, t.t, r.r parity 0/1, s.s
struct BcgParts {
    double *base;
    int G;
    bool slices;
    __device__ double *rho(int k) const { return base + (size_t)(k & 1) * G; }
    __host__ __device__ double *rv() const { return base + (size_t)2 * G; }
    __host__ __device__ double *ts() const { return base + (size_t)3 * G; }
    __host__ __device__ double *tt() const { return base + (size_t)4 * G; }
    __device__ double *rr(int k) const { return base + (size_t)(5 + (k & 1)) * G; }
    __device__ double *ss() const { return base + (size_t)7 * G; }
};

// The sums of several partial arrays in one pass and one block reduction (one
// at a time, each costs its own two barriers and chain of loads, ~1 us: six of
// them were half of the direction kernel's 8 us).
template <int N>
__device__ inline void totals(const BcgParts &P, const double *const (&p)[N], double (&v)[N]) {
    krylov_sums<kT>(P.slices, [&](int i) { return p[i]; }, P.G, v);
}
__device__ inline int my_slice() { return (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6); }

// x0 given: r = b - A x, rhat = r;
// partials r.r and rhat.r for iteration k0 - 1
__global__ __launch_bounds__(kT) void bcg_init_kernel(Sell<double> A, int k0, const double *__restrict__ b,
                                                      const double *__restrict__ x, double *__restrict__ r,
                                                      double *__restrict__ rhat, BcgParts P) {
    krylov_rows<kT, 2, false, double, double>(
        A, P.slices, P.G, [&](int32_t j) { return x[j]; },
        [&](int32_t i, double s, double *v) {
            const double ri = b[i] - s;
            r[i] = ri;
            rhat[i] = ri;
            v[0] += ri * ri;
            v[1] += ri * ri;
        },
        [&](int i) { return i ? P.rho(k0 - 1) : P.rr(k0 - 1); });
}
// the same for x = 0
__global__ __launch_bounds__(kT) void bcg_init_zero_kernel(int32_t n, int k0, const double *__restrict__ b,
                                                           double *__restrict__ x, double *__restrict__ r,
                                                           double *__restrict__ rhat, BcgParts P) {
    double v[2] = {0.0, 0.0};
    GSB(i, n) {
        const double ri = b[i];
        x[i] = 0.0;
        r[i] = ri;
        rhat[i] = ri;
        v[0] += ri * ri;
        v[1] += ri * ri;
    }
    krylov_put<kT, 2>(P.slices, [&](int i) { return i ? P.rho(k0 - 1) : P.rr(k0 - 1); }, my_slice(), v);
}

__global__ __launch_bounds__(kT) void bcg_start_kernel(BcgParts P, PcgState *st, double rtol, int k0,
                                                       int *host_done) {
    double v[1];
    totals(P, {P.rr(k0 - 1)}, v);
    const double rr = v[0];
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        if (k0 == 0) st->bnorm2 = rr;
        st->tol2 = rtol * rtol * rr;
        st->rr = rr;
        st->iter = k0;
        st->host_done = host_done;
        st->done = st->converged = 0;
        if (rr == 0.0) krylov_done(st, 1, rr);
    }
}

// convergence test on r_{k-1}, then the search direction p
__global__ __launch_bounds__(kT) void bcg_direction_kernel(int32_t n, int k, int k0, const double *__restrict__ r,
                                                           double *__restrict__ p, const double *__restrict__ v,
                                                           BcgParts P, PcgState *st, int update) {
    if (st->done) return;
    // those of the last iteration are read (and not used) before there is one
    double w[6];
    totals(P, {P.rr(k - 1), P.rho(k - 1), P.rho(k - 2), P.rv(), P.ts(), P.tt()}, w);
    const double rr = w[0], rho = w[1];
    const bool conv = rr <= st->tol2;
    if (conv || rho == 0.0 || !(rr == rr)) {  // converged, breakdown (rhat orthogonal to r) or NaN
        if (blockIdx.x == 0 && threadIdx.x == 0) krylov_done(st, conv ? 1 : 0, rr);
        return;
    }
    if (!update) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->rr = rr;
        return;
    }
    if (k == k0) {
        GSB(i, n) p[i] = r[i];
        return;
    }
    const double rho_prev = w[2];
    const double alpha = rho_prev / w[3];
    const double omega = w[4] / w[5];
    const double beta = (rho / rho_prev) * (alpha / omega);
    GSB(i, n) p[i] = r[i] + beta * (p[i] - omega * v[i]);
}

// y = A x with the partials of w . y into parts (and of y . y into parts2).
// LOCAL: each XCD takes a run of the rows; the partials go to the places of their
// slices either way.
template <bool SPLIT, bool LOCAL>
__global__ __launch_bounds__(SPLIT ? kSplitThreads : kT) void bcg_spmv_dot_kernel(Sell<double> A, const double *__restrict__ x,
                                                          double *__restrict__ y, const double *__restrict__ w,
                                                          BcgParts P, double *__restrict__ parts,
                                                          double *__restrict__ parts2, const PcgState *st) {
    if (st->done) return;
    auto f = [&](int32_t j) { return x[j]; };
    auto row = [&](int32_t i, double yi, double *v) {
        y[i] = yi;
        v[0] += w[i] * yi;
        v[1] += yi * yi;
    };
    auto put = [&](int i) { return i ? parts2 : parts; };
    if constexpr (SPLIT) {
        const int32_t i = split_row<kSplitThreads, LOCAL>();
        const double s = lane_row(A, i, f).template sum<double, 1>([](double t) { return t; });
        split_rows<kSplitThreads, 2, LOCAL, false>(A.n, P.G, i, s, row, put);
    } else {
        krylov_rows<kT, 2, false, double, double>(A, false, P.G, f, row, put);
    }
}

// s = r - alpha v and the partials of s.s
__global__ __launch_bounds__(kT) void bcg_s_kernel(int32_t n, int k, const double *__restrict__ r,
                                                   const double *__restrict__ v, double *__restrict__ s, BcgParts P,
                                                   const PcgState *st) {
    if (st->done) return;
    double c[2];
    totals(P, {P.rho(k - 1), P.rv()}, c);
    const double alpha = c[0] / c[1];
    double w[1] = {0.0};
    GSB(i, n) {
        const double si = r[i] - alpha * v[i];
        s[i] = si;
        w[0] += si * si;
    }
    krylov_put<kT, 1>(P.slices, [&](int) { return P.ss(); }, my_slice(), w);
}

// x += alpha phat + omega shat, r = s - omega t; partials r.r and rhat.r.
// When |s|^2 already meets the tolerance, x += alpha phat and r = s: the next
// direction kernel finds the solve converged.  Asked here, behind the second
// product, because a kernel of its own for the question took 3 us of every
// iteration.
__global__ __launch_bounds__(kT) void bcg_update_kernel(int32_t n, int k, const double *__restrict__ phat,
                                                        const double *__restrict__ shat,
                                                        const double *__restrict__ s, const double *__restrict__ t,
                                                        const double *__restrict__ rhat, double *__restrict__ x,
                                                        double *__restrict__ r, BcgParts P, PcgState *st) {
    if (st->done) return;
    double c[5];
    totals(P, {P.rho(k - 1), P.rv(), P.tt(), P.ts(), P.ss()}, c);
    const double alpha = c[0] / c[1], tt = c[2];
    const bool half = c[4] <= st->tol2;
    const double omega = tt > 0.0 ? c[3] / tt : 0.0;
    double v[2] = {0.0, 0.0};
    GSB(i, n) {
        const double xi = x[i], step = fma(alpha, phat[i], omega * shat[i]);
        x[i] = half ? fma(alpha, phat[i], xi) : xi + step;
        const double ri = half ? s[i] : s[i] - omega * t[i];
        r[i] = ri;
        v[0] += ri * ri;
        v[1] += rhat[i] * ri;
    }
    krylov_put<kT, 2>(P.slices, [&](int i) { return i ? P.rho(k) : P.rr(k); }, my_slice(), v);
    if (threadIdx.x == 0 && blockIdx.x == 0) st->iter = k + 1;
}

}  // namespace

static BcgParts bcg_parts(const BcgWork &W) { return BcgParts{W.parts, W.shape.G, W.shape.split}; }

#define BLAUNCH(blocks, kern, ...)                                                                           \
    do {                                                                                                     \
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(kT), 0, s, __VA_ARGS__);                                 \
        VAG_HIP(hipGetLastError());                                                                          \
    } while (0)
#define BROWS(kern, ...)                                                                                      \
    VAG_ROWS_LAUNCH(W.shape, hipLaunchKernelGGL((W.local ? kern<SPLIT, SPLIT> : kern<SPLIT, false>),          \
                                                dim3(ks.row_blocks), dim3(threads), 0, s, __VA_ARGS__))

void launch_bcg_init(hipStream_t s, Sell<double> A, bool zero_x, int k0, const double *b, double *x, double *r,
                     double *rhat, const BcgWork &W) {
    const BcgParts P = bcg_parts(W);
    if (zero_x)
        BLAUNCH(W.shape.vec_blocks, bcg_init_zero_kernel, A.n, k0, b, x, r, rhat, P);
    else
        BLAUNCH(W.shape.vec_blocks, bcg_init_kernel, A, k0, b, x, r, rhat, P);
}
void launch_bcg_start(hipStream_t s, int32_t n, const BcgWork &W, PcgState *st, double rtol, int k0, int *host_done) {
    BLAUNCH(1, bcg_start_kernel, bcg_parts(W), st, rtol, k0, host_done);
}
void launch_bcg_direction(hipStream_t s, int32_t n, int k, int k0, const double *r, double *p, const double *v,
                          const BcgWork &W, PcgState *st, bool update) {
    const BcgParts P = bcg_parts(W);
    BLAUNCH(W.shape.vec_blocks, bcg_direction_kernel, n, k, k0, r, p, v, P, st, update ? 1 : 0);
}
void launch_bcg_spmv_v(hipStream_t s, Sell<double> A, const double *phat, double *v, const double *rhat,
                       const BcgWork &W, const PcgState *st) {
    const BcgParts P = bcg_parts(W);
    BROWS(bcg_spmv_dot_kernel, A, phat, v, rhat, P, P.rv(), (double *)nullptr, st);
}
void launch_bcg_s(hipStream_t s, int32_t n, int k, const double *r, const double *v, double *sv, const BcgWork &W,
                  const PcgState *st) {
    const BcgParts P = bcg_parts(W);
    BLAUNCH(W.shape.vec_blocks, bcg_s_kernel, n, k, r, v, sv, P, st);
}
void launch_bcg_spmv_t(hipStream_t s, Sell<double> A, const double *shat, double *t, const double *sv, const BcgWork &W,
                       const PcgState *st) {
    const BcgParts P = bcg_parts(W);
    BROWS(bcg_spmv_dot_kernel, A, shat, t, sv, P, P.ts(), P.tt(), st);
}
void launch_bcg_update(hipStream_t s, int32_t n, int k, const double *phat, const double *shat, const double *sv,
                       const double *t, const double *rhat, double *x, double *r, const BcgWork &W, PcgState *st) {
    const BcgParts P = bcg_parts(W);
    BLAUNCH(W.shape.vec_blocks, bcg_update_kernel, n, k, phat, shat, sv, t, rhat, x, r, P, st);
}

}  // namespace vag
