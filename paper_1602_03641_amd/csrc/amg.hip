// Aggregation AMG for the SPD system of eq eqschur, set up on the device at
// every solve (the matrix values change with the permeabilities).
//
// Coarsening (one level):
//   strength   j is a strong neighbour of i if |a_ij| >= theta sqrt(|a_ii a_jj|)
//   roots      a distance-2 maximal independent set of the strength graph,
//              found by rounds of 2-hop max propagation of (state, priority)
//              keys, the priority a bijective hash of the row index; later
//              rounds exit at once when nothing is left undecided (the host
//              polls)
//   aggregates each root starts one; other nodes join their strongest root
//              neighbour, then the strongest already-aggregated neighbour
//   P          piecewise-constant interpolation (one 1 per row)
//   A_c        = P^T A P, one wavefront per coarse row: the rows of A P
//              (each fine row's entries collapsed per aggregate) of the
//              aggregate's members are gathered as (coarse column, gather
//              ordinal) keys with their values in LDS, bitonic-sorted, and
//              each coarse entry sums its candidates in gather order, so the
//              coarse matrix is bitwise reproducible
// Smoother: l1-Jacobi, M = diag(sum_j |a_ij|), convergent for any SPD matrix.
// Cycle: symmetric V-cycle (one pre- and one post-sweep on the finest level,
// `sweeps` of each on the coarser ones), the coarsest level
// solved by a dense inverse formed on the device by Gauss-Jordan elimination.
#include <algorithm>

#include "amg.h"
#include "reduce.h"
#include "sell.h"

namespace vag {

constexpr int kAT = 256;
constexpr int kCap = 8192;  // candidate entries per coarse row held in LDS

#define GS(i, n) \
    for (int64_t i = (int64_t)xcd_block() * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// full grid for the grid-stride kernels (no reduction partials)
static inline unsigned gridv(int64_t n) {
    const int64_t b = (n + kAT - 1) / kAT;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 1 << 20));
}

// A bijection of [0, 2^30): odd multipliers and right xor-shifts are each
// invertible modulo 2^30, so distinct rows get distinct priorities.
__device__ inline uint32_t perm30(uint32_t x) {
    constexpr uint32_t kM = (1u << 30) - 1;
    x &= kM;
    x = (x * 0x2c1b3c6du) & kM;
    x ^= x >> 15;
    x = (x * 0x297a2d39u) & kM;
    x ^= x >> 13;
    return x;
}
// MIS keys: state in the top two bits (2 root, 1 undecided, 0 out), the
// row's priority below
__device__ inline int rank_of(uint32_t t) { return (int)(t >> 30); }

// diag and l1-Jacobi inverse
__global__ __launch_bounds__(kAT) void amg_diag_kernel(Sell<double> A, double *__restrict__ diag,
                                                       double *__restrict__ dinv) {
    GS(i, A.n) {
        double d = 0.0, l1 = 0.0, v[kSlots];
        int32_t c[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t q) {
                v[j] = A.val[q];
                c[j] = A.col[q];
            },
            [&](int j, int64_t) {
                if (c[j] == i) d += v[j];
                l1 += fabs(v[j]);
            });
        diag[i] = d;
        dinv[i] = 1.0 / l1;
    }
}

// scol[q] = column of entry q if it is a strong off-diagonal coupling, else
// the row itself (so the MIS passes gather without branches: a row's own key
// never changes a maximum that already includes it); the keys' start, and
// every counter of the level cleared (one launch where six were: on a small
// level a launch is its whole time)
__global__ __launch_bounds__(kAT) void strength_kernel(Sell<double> A, const double *__restrict__ diag, double theta,
                                                       int32_t *__restrict__ scol, CoarsenInit I) {
    GS(k, I.nundecided) I.undecided[k] = 0;
    GS(k, 64) I.counters[k] = 0;
    GS(i, (int64_t)A.n + 1) I.cnt[i] = I.cursor[i] = 0;
    GS(i, A.n) {
        const double di = diag[i];
        double v[kSlots], dj[kSlots];
        int32_t c[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t q) {
                v[j] = A.val[q];
                c[j] = A.col[q];
                dj[j] = diag[c[j]];
            },
            [&](int j, int64_t q) {
                const double a = fabs(v[j]);
                scol[q] = c[j] != i && a != 0.0 && a >= theta * sqrt(fabs(di * dj[j])) ? c[j] : (int32_t)i;
            });
        I.T[i] = (1u << 30) | perm30((uint32_t)i);
        I.T1[i] = 1u << 30;  // rank 1: computed in the first round
    }
}

// max of key[] over row i and its strong neighbours, four gathers in flight
__device__ inline uint32_t strong_max(const int64_t *__restrict__ ptr, const int32_t *__restrict__ scol, int32_t i,
                                      const uint32_t *__restrict__ key) {
    const int64_t b1 = ptr[(i >> 6) + 1];
    int64_t q = ptr[i >> 6] + (i & 63);
    uint32_t m0 = key[i], m1 = 0, m2 = 0, m3 = 0;
    for (; q + 192 < b1; q += 256) {
        m0 = max(m0, key[scol[q]]);
        m1 = max(m1, key[scol[q + 64]]);
        m2 = max(m2, key[scol[q + 128]]);
        m3 = max(m3, key[scol[q + 192]]);
    }
    for (; q < b1; q += 64) m0 = max(m0, key[scol[q]]);
    return max(max(m0, m1), max(m2, m3));
}

// Per-round counts of undecided rows, spread over kCntSlots counters 128 bytes
// apart: device-wide atomics on one address serialise, and thousands of
// blocks adding to a single counter cost more than the round itself.
__device__ inline bool any_count(const int *__restrict__ c) {
    const int lane = threadIdx.x & 63;
    const int v = lane < kCntSlots ? c[lane * kCntStride] : 0;
    return __ballot(v != 0) != 0;
}

// Tout[i] = max of T over {i} and its strong neighbours, recomputed only
// where the previous round's maximum had rank 1 (an undecided row among
// them).  Rank 0: every row of the set was decided, and decided keys never
// change, so the value is still exact.  Rank 2: a root among them, which stays
// a root, so the maximum still has rank 2; the selection asks of a maximum
// only whether it has rank 2 or, having rank 1, equals an undecided row's own
// key, so its decisions are those of the full recomputation.  The later
// rounds then touch only the rows next to the undecided ones.
__global__ __launch_bounds__(kAT) void mis_max_kernel(int32_t n, const int64_t *__restrict__ ptr,
                                                      const int32_t *__restrict__ scol, const uint32_t *__restrict__ Tin,
                                                      uint32_t *__restrict__ Tout, const int *__restrict__ active,
                                                      int round, int *progress) {
    const bool over = active && !any_count(active);
    if (blockIdx.x == 0 && threadIdx.x == 0) host_put(progress, over ? kMisRounds + 1 : round + 1);
    if (over) return;
    GS(i, n) {
        if (rank_of(Tout[i]) != 1) continue;
        Tout[i] = strong_max(ptr, scol, (int32_t)i, Tin);
    }
}

// second hop, then the decision of undecided nodes
__global__ __launch_bounds__(kAT) void mis_select_kernel(int32_t n, int hops, const int64_t *__restrict__ ptr,
                                                         const int32_t *__restrict__ scol,
                                                         const uint32_t *__restrict__ T1, uint32_t *__restrict__ T,
                                                         int *__restrict__ undecided, const int *__restrict__ active) {
    __shared__ int wc[kAT / 64];
    if (active && !any_count(active)) return;  // uniform over the block: every wave reads the same counters
    int cnt = 0;
    GS(i, n) {
        const uint32_t own = T[i];
        if (rank_of(own) != 1) continue;
        // two hops: the maximum over the neighbours of the one-hop maxima; one
        // hop: the one-hop maximum itself
        const uint32_t m = hops == 2 ? strong_max(ptr, scol, (int32_t)i, T1) : T1[i];
        if (m == own)
            T[i] = (own & ((1u << 30) - 1)) | (2u << 30);  // root
        else if (rank_of(m) == 2)
            T[i] = own & ((1u << 30) - 1);  // a root lies within distance 2
        else
            ++cnt;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if ((threadIdx.x & 63) == 0) wc[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < kAT / 64; ++w) t += wc[w];
        if (t) atomicAdd(undecided + (blockIdx.x % kCntSlots) * kCntStride, t);  // integer count, order-independent
    }
}

// roots (and nodes left undecided) flagged 1
__global__ __launch_bounds__(kAT) void mis_flag_kernel(int32_t n, const uint32_t *__restrict__ T,
                                                       int32_t *__restrict__ flag) {
    GS(i, n) flag[i] = rank_of(T[i]) >= 1 ? 1 : 0;
}

// The strongest of row i's strong neighbours j (ties: the least j) with
// mark[j] set, or -1; s_ij = |a_ij| / sqrt(|a_ii a_jj|).  The rows' strong
// columns are at hand (scol; a weak slot holds the row itself, whose mark is
// not set), so the values are read only where a neighbour is marked: both
// passes together 69 us at 64^3 and 580 us at 128^3 while they tested the
// strength of every entry again, now 48 and 284.
template <class Mark>
__device__ inline int32_t strongest(const Sell<double> &A, const double *__restrict__ diag,
                                    const int32_t *__restrict__ scol, int64_t i, Mark mark) {
    const double di = diag[i];
    double best = -1.0;
    int32_t bj = -1, c[kSlots];
    bool m[kSlots];
    row_slots(
        A.ptr, i,
        [&](int j, int64_t q) {
            c[j] = scol[q];
            m[j] = mark(c[j]);
        },
        [&](int j, int64_t q) {
            if (!m[j]) return;
            const double s = fabs(A.val[q]) / sqrt(fabs(di * diag[c[j]]));
            if (s > best || (s == best && c[j] < bj)) {
                best = s;
                bj = c[j];
            }
        });
    return bj;
}
__global__ __launch_bounds__(kAT) void agg_pass1_kernel(Sell<double> A, const double *__restrict__ diag,
                                                        const int32_t *__restrict__ scol,
                                                        const int32_t *__restrict__ root, const int32_t *__restrict__ rid,
                                                        int32_t *__restrict__ agg1) {
    GS(i, A.n) {
        if (root[i]) {
            agg1[i] = rid[i];
            continue;
        }
        const int32_t bj = strongest(A, diag, scol, i, [&](int32_t j) { return root[j] != 0; });
        agg1[i] = bj >= 0 ? rid[bj] : -1;
    }
}

__global__ __launch_bounds__(kAT) void agg_pass2_kernel(Sell<double> A, const double *__restrict__ diag,
                                                        const int32_t *__restrict__ scol,
                                                        const int32_t *__restrict__ agg1, int32_t *__restrict__ agg,
                                                        int32_t *__restrict__ lonely) {
    GS(i, A.n) {
        int32_t a = agg1[i];
        if (a < 0) {
            const int32_t bj = strongest(A, diag, scol, i, [&](int32_t j) { return agg1[j] >= 0; });
            if (bj >= 0) a = agg1[bj];
        }
        agg[i] = a;
        lonely[i] = a < 0 ? 1 : 0;
    }
}

__global__ __launch_bounds__(kAT) void count_kernel(int32_t n, const int32_t *__restrict__ agg,
                                                    int32_t *__restrict__ cnt) {
    GS(i, n) atomicAdd(&cnt[agg[i]], 1);
}
__global__ __launch_bounds__(kAT) void members_fill_kernel(int32_t n, const int32_t *__restrict__ agg,
                                                           const int32_t *__restrict__ ptr, int32_t *__restrict__ cursor,
                                                           int32_t *__restrict__ rows) {
    GS(i, n) {
        const int32_t a = agg[i];
        rows[ptr[a] + atomicAdd(&cursor[a], 1)] = (int32_t)i;
    }
}
// members in ascending row order: the rank of each member is the number of
// smaller members (one wavefront per aggregate; atomic fill order is arbitrary)
__global__ __launch_bounds__(kAT) void members_rank_kernel(int32_t nc, const int32_t *__restrict__ ptr,
                                                           const int32_t *__restrict__ tmp, int32_t *__restrict__ rows) {
    const int lane = threadIdx.x & 63;
    const int64_t w0 = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t I = w0; I < nc; I += nw) {
        const int32_t b = ptr[I], e = ptr[I + 1];
        for (int32_t t = b + lane; t < e; t += 64) {
            const int32_t v = tmp[t];
            int32_t rank = 0;
            for (int32_t u = b; u < e; ++u) rank += tmp[u] < v;
            rows[b + rank] = v;
        }
    }
}

// Where a scan goes: out[k] the sum before k and out[n] the total; or, for the
// flagged k alone, agg[k] = *base + the sum before k.  host (pinned): the total.
struct ScanTo {
    int32_t *out, *agg;
    const int32_t *base;
    int *host;
    __device__ inline void put(int64_t k, int32_t in, int32_t run) const {
        if (out) out[k] = run;
        else if (in) agg[k] = *base + run;
    }
    __device__ inline void total(int64_t n, int32_t t) const {
        if (out) out[n] = t;
        if (host) host_put(host, t);
    }
};
// exclusive scan of n ints in one block, a run of them per thread
__global__ __launch_bounds__(1024) void scan_int_kernel(int32_t n, const int32_t *__restrict__ in,
                                                        ScanTo to) {
    __shared__ int32_t part[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int32_t chunk = (n + 1023) / 1024;
    const int32_t lo = min(n, t * chunk), hi = min(n, lo + chunk);
    int32_t s = 0;
    for (int32_t k = lo; k < hi; ++k) s += in[k];
    int32_t incl = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) part[w] = incl;
    __syncthreads();
    int32_t run = incl - s;
    for (int k = 0; k < w; ++k) run += part[k];
    if (t == 1023) to.total(n, run + s);
    for (int32_t k = lo; k < hi; ++k) {
        const int32_t v = in[k];
        to.put(k, v, run);
        run += v;
    }
}

// multi-block exclusive scan of n ints: block sums, one-block
// scan of the block sums, then per-block scan with offsets
constexpr int kScanItems = 4;
__global__ __launch_bounds__(256) void scan_sums_kernel(int32_t n, const int32_t *__restrict__ in,
                                                        int32_t *__restrict__ sums) {
    __shared__ int32_t w[4];
    const int64_t base = (int64_t)blockIdx.x * 256 * kScanItems;
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + (int64_t)k * 256 + threadIdx.x;
        if (i < n) s += in[i];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = w[0] + w[1] + w[2] + w[3];
}
__global__ __launch_bounds__(256) void scan_apply_kernel(int32_t n, const int32_t *__restrict__ in,
                                                         const int32_t *__restrict__ offs, ScanTo to) {
    __shared__ int32_t wsum[4];
    const int64_t base = (int64_t)blockIdx.x * 256 * kScanItems + (int64_t)threadIdx.x * kScanItems;
    int32_t v[kScanItems];
    int32_t t = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        t += v[k];
    }
    // inclusive scan of t over the block
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int32_t incl = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int32_t off = offs[blockIdx.x];
    for (int k = 0; k < wv; ++k) off += wsum[k];
    int32_t run = off + incl - t;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) to.put(base + k, v[k], run);
        run += v[k];
    }
    if (base + kScanItems >= n && base < n) to.total(n, run);  // the thread holding the last element
}

// ---------------------------------------------------------------------------
// Galerkin coarse operator, one wavefront per coarse row
// ---------------------------------------------------------------------------
// Row i of A P (P = aggregate indicator): the distinct aggregates of the row's
// columns, in increasing order, each with the sum of its entries (in entry
// order); the nonzero sums go to the row's first apn[i] slots of (apJ, apv).
// The lanes of a wave scan slot k together, so the passes are coalesced, eight
// slots' aggregates read ahead (64^3: 73 us after a pass of 29 us that wrote
// them out, now 59; 128^3: 331 and 150, now 294).  A
// row with more than kSet distinct aggregates is appended to the spill list
// and collapsed by ap_spill_kernel instead.
constexpr int kSet = 16;
__global__ __launch_bounds__(kAT) void ap_collapse_kernel(Sell<double> A, const int32_t *__restrict__ agg,
                                                          int32_t *__restrict__ apJ, double *__restrict__ apv,
                                                          int32_t *__restrict__ apn, int32_t *__restrict__ spill,
                                                          int *__restrict__ nspill) {
    GS(i, A.n) {
        const int64_t b0 = A.ptr[i >> 6] + (i & 63);
        int32_t J[kSet];
        double v[kSet];
        int cnt = 0;
        bool over = false;
#pragma unroll
        for (int t = 0; t < kSet; ++t) {
            J[t] = INT32_MAX;
            v[t] = 0.0;
        }
        double av[kSlots];
        int32_t cv[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t q) {
                av[j] = A.val[q];
                cv[j] = agg[A.col[q]];
            },
            [&](int j, int64_t) {
                const double a = av[j];
                if (a == 0.0 || over) return;
                const int32_t c = cv[j];
                bool found = false;
#pragma unroll
                for (int t = 0; t < kSet; ++t)
                    if (J[t] == c) {
                        v[t] += a;
                        found = true;
                    }
                if (!found) {
                    if (cnt == kSet) {
                        over = true;
                    } else {
#pragma unroll
                        for (int t = 0; t < kSet; ++t)
                            if (t == cnt) {
                                J[t] = c;
                                v[t] = a;
                            }
                        ++cnt;
                    }
                }
            });
        if (over) {
            spill[atomicAdd(nspill, 1)] = (int32_t)i;  // list order is irrelevant: rows are independent
            continue;
        }
        // ascending aggregate order (selection of the next larger key)
        int64_t out = b0;
        int32_t last = -1;
        int written = 0;
        for (int k = 0; k < cnt; ++k) {
            int32_t jm = INT32_MAX;
            double vm = 0.0;
#pragma unroll
            for (int t = 0; t < kSet; ++t)
                if (J[t] > last && J[t] < jm) {
                    jm = J[t];
                    vm = v[t];
                }
            last = jm;
            if (vm == 0.0) continue;
            apJ[out] = jm;
            apv[out] = vm;
            out += 64;
            ++written;
        }
        apn[i] = written;
    }
}

// The spilled rows of ap_collapse_kernel, one wavefront per row: the row's
// entries as keys (aggregate, slot) sorted in LDS, then one sum per run of
// equal aggregates in slot order (the order of the fast path).  Rows with more
// than CAP entries fall back to repeated minimum extraction by one lane.
template <int CAP>
__global__ __launch_bounds__(64) void ap_spill_kernel(Sell<double> A, const int32_t *__restrict__ agg,
                                                      int32_t *__restrict__ apJ, double *__restrict__ apv,
                                                      int32_t *__restrict__ apn, const int32_t *__restrict__ spill,
                                                      const int *__restrict__ nspill) {
    __shared__ uint64_t key[CAP];
    const int lane = threadIdx.x;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int ns = *nspill;
    for (int it = blockIdx.x; it < ns; it += gridDim.x) {
        const int32_t r = spill[it];
        const int64_t b0 = A.ptr[r >> 6] + (r & 63);
        const int w = (int)((A.ptr[(r >> 6) + 1] - A.ptr[r >> 6]) >> 6);
        int m = 0;
        for (int k0 = 0; k0 < w && m <= CAP; k0 += 64) {
            const int k = k0 + lane;
            bool keep = false;
            uint64_t kv = 0;
            if (k < w) {
                const int64_t q = b0 + (int64_t)k * 64;
                if (A.val[q] != 0.0) {
                    keep = true;
                    kv = ((uint64_t)(uint32_t)agg[A.col[q]] << 32) | (uint64_t)(uint32_t)k;
                }
            }
            const uint64_t mask = __ballot(keep);
            const int off = __popcll(mask & below);
            if (keep && m + off < CAP) key[m + off] = kv;
            m += __popcll(mask);
        }
        if (m > CAP) {
            if (lane == 0) {
                int32_t last = -1;
                int written = 0;
                int64_t out = b0;
                for (;;) {
                    int32_t jm = INT32_MAX;
                    for (int k = 0; k < w; ++k) {
                        const int64_t q = b0 + (int64_t)k * 64;
                        const int32_t c = agg[A.col[q]];
                        if (c > last && c < jm && A.val[q] != 0.0) jm = c;
                    }
                    if (jm == INT32_MAX) break;
                    double sum = 0.0;
                    for (int k = 0; k < w; ++k) {
                        const int64_t q = b0 + (int64_t)k * 64;
                        const double a = A.val[q];
                        if (a != 0.0 && agg[A.col[q]] == jm) sum += a;
                    }
                    last = jm;
                    if (sum == 0.0) continue;
                    apJ[out] = jm;
                    apv[out] = sum;
                    out += 64;
                    ++written;
                }
                apn[r] = written;
            }
            __syncthreads();
            continue;
        }
        int mp = 1;
        while (mp < m) mp <<= 1;
        for (int k = m + lane; k < mp; k += 64) key[k] = ~0ull;
        __syncthreads();
        for (int k = 2; k <= mp; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = lane; i < mp; i += 64) {
                    const int p = i ^ j;
                    if (p > i) {
                        const uint64_t a = key[i], b = key[p];
                        const bool up = (i & k) == 0;
                        if ((a > b) == up) {
                            key[i] = b;
                            key[p] = a;
                        }
                    }
                }
                __syncthreads();
            }
        // runs of equal aggregates: lane-contiguous chunks, nonzero sums ranked by a wave scan
        const int C = (m + 63) / 64;
        const int lo = min(m, lane * C), hi = min(m, lo + C);
        int nh = 0;
        for (int t = lo; t < hi; ++t) {
            if (!(t == 0 || (key[t] >> 32) != (key[t - 1] >> 32))) continue;
            const uint32_t Jt = (uint32_t)(key[t] >> 32);
            double s = 0.0;
            for (int u = t; u < m && (uint32_t)(key[u] >> 32) == Jt; ++u) s += A.val[b0 + (int64_t)(uint32_t)key[u] * 64];
            nh += s != 0.0;
        }
        int incl = nh;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        int rank = incl - nh;
        for (int t = lo; t < hi; ++t) {
            if (!(t == 0 || (key[t] >> 32) != (key[t - 1] >> 32))) continue;
            const uint32_t Jt = (uint32_t)(key[t] >> 32);
            double s = 0.0;
            for (int u = t; u < m && (uint32_t)(key[u] >> 32) == Jt; ++u) s += A.val[b0 + (int64_t)(uint32_t)key[u] * 64];
            if (s == 0.0) continue;
            apJ[b0 + (int64_t)rank * 64] = (int32_t)Jt;
            apv[b0 + (int64_t)rank * 64] = s;
            ++rank;
        }
        if (lane == 63) apn[r] = incl;
        __syncthreads();
    }
}

// Galerkin coarse row I, one wavefront: the collapsed entries (apn[r] of
// them) of the aggregate's rows r are gathered as (coarse column, value) in
// gather order, one member row per lane; the distinct columns are found with
// an LDS hash set, ranked (each rank counts the smaller columns), and each
// column sums its candidates in gather order (all lanes read candidate k
// together), so the coarse matrix is bitwise reproducible.  mode 0:
// rowlen[I] = number of coarse columns, big[I] = 1 for a row this kernel
// cannot hold, appended to biglist (*nbig of them); mode 1: write the row
// (SELL).  Bound by the latency of the chains of LDS reads, 9 wavefronts on a
// CU (52 k rows of a 128^3 mesh: 560 us in mode 1 with one candidate per turn,
// now 346).
constexpr int kGalCand = 1024, kGalHash = 512, kGalDistinct = 256, kGalBatch = 8;
__global__ __launch_bounds__(64) void galerkin_hash_kernel(Sell<double> A, const int32_t *__restrict__ Jcol,
                                                           const double *__restrict__ apv,
                                                           const int32_t *__restrict__ apn,
                                                           const int32_t *__restrict__ mptr,
                                                           const int32_t *__restrict__ mrows, int32_t nc, int mode,
                                                           int32_t *__restrict__ big, int32_t *__restrict__ biglist,
                                                           int *__restrict__ nbig, int32_t *__restrict__ rowlen,
                                                           const int64_t *__restrict__ cptr,
                                                           int32_t *__restrict__ ccol, double *__restrict__ cval) {
    __shared__ __align__(16) int32_t cj[kGalCand];
    __shared__ __align__(16) double cv[kGalCand];
    __shared__ int32_t hs[kGalHash];
    __shared__ int32_t dist[kGalDistinct];
    __shared__ int32_t sorted[kGalDistinct];
    const int32_t I = blockIdx.x;
    const int lane = threadIdx.x;
    if (I >= nc) return;
    if (mode == 1 && big[I]) return;
    for (int k = lane; k < kGalHash; k += 64) hs[k] = -1;
    // gather
    int m = 0;
    bool over = false;
    const int32_t t1 = mptr[I + 1];
    for (int32_t t0 = mptr[I]; t0 < t1; t0 += 64) {
        const int32_t t = t0 + lane;
        int c = 0;
        int64_t b = 0;
        if (t < t1) {
            const int32_t r = mrows[t];
            b = A.ptr[r >> 6] + (r & 63);
            c = apn[r];
        }
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        const int tot = __shfl(incl, 63, 64);
        if (m + tot > kGalCand) {
            over = true;
            break;
        }
        const int off = m + incl - c;
        for (int k0 = 0; k0 < c; k0 += 4) {  // four entries' loads in flight
            int32_t J[4];
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t q = b + (int64_t)min(k0 + u, c - 1) * 64;
                J[u] = Jcol[q];
                v[u] = apv[q];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u < c) {
                    cj[off + k0 + u] = J[u];
                    cv[off + k0 + u] = v[u];
                }
        }
        m += tot;
    }
    __syncthreads();
    // distinct columns: an LDS hash set (linear probing); a set that grows
    // past kGalDistinct sends the row to the sorting kernel
    bool full = false;
    if (!over) {
        for (int k = lane; k < m; k += 64) {
            const int32_t J = cj[k];
            uint32_t h = ((uint32_t)J * 2654435761u) & (kGalHash - 1);
            for (int probe = 0; probe < kGalHash; ++probe) {
                const int32_t prev = atomicCAS(&hs[h], -1, J);
                if (prev == -1 || prev == J) break;
                h = (h + 1) & (kGalHash - 1);
            }
        }
    }
    __syncthreads();
    int nd = 0;
    if (!over) {
        // compact the occupied slots
        for (int k0 = 0; k0 < kGalHash; k0 += 64) {
            const int32_t J = hs[k0 + lane];
            const uint64_t mask = __ballot(J >= 0);
            const int below = __popcll(mask & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
            const int base = nd;
            if (J >= 0 && base + below < kGalDistinct) dist[base + below] = J;
            nd += __popcll(mask);
        }
        full = nd > kGalDistinct;
    }
    if (over || full) {
        if (mode == 0 && lane == 0) {
            big[I] = 1;
            biglist[atomicAdd(nbig, 1)] = I;  // list order is irrelevant: rows are independent
        }
        return;
    }
    if (mode == 0 && lane == 0) big[I] = 0;
    // candidates that no column takes, up to a multiple of kGalBatch
    const int mp = (m + kGalBatch - 1) / kGalBatch * kGalBatch;
    if (m + lane < mp) {
        cj[m + lane] = -2;
        cv[m + lane] = 0.0;
    }
    __syncthreads();
    // rank sort of the distinct columns
    for (int i = lane; i < nd; i += 64) {
        const int32_t J = dist[i];
        int rank = 0;
#pragma unroll 8
        for (int u = 0; u < nd; ++u) rank += dist[u] < J;
        sorted[rank] = J;
    }
    if (mode == 0) {
        if (lane == 0) rowlen[I] = nd;
        return;
    }
    __syncthreads();
    // sums in gather order; lane owns sorted columns lane, lane + 64, ...
    constexpr int kOwn = kGalDistinct / 64;
    int32_t own[kOwn];
    double sum[kOwn];
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
        own[o] = (lane + 64 * o < nd) ? sorted[lane + 64 * o] : -1;
        sum[o] = 0.0;
    }
    const int nown = (nd + 63) / 64;
    // a batch of candidates per turn: one at a time, each waited for its LDS read
    for (int k = 0; k < mp; k += kGalBatch) {
        int32_t J[kGalBatch];
        double v[kGalBatch];
#pragma unroll
        for (int u = 0; u < kGalBatch; ++u) {
            J[u] = cj[k + u];
            v[u] = cv[k + u];
        }
#pragma unroll
        for (int o = 0; o < kOwn; ++o)
            if (o < nown)
#pragma unroll
                for (int u = 0; u < kGalBatch; ++u)
                    if (own[o] == J[u]) sum[o] += v[u];
    }
    const int64_t base = cptr[I >> 6] + (I & 63);
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
        const int k = lane + 64 * o;
        if (k < nd) {
            ccol[base + (int64_t)k * 64] = own[o];
            cval[base + (int64_t)k * 64] = sum[o];
        }
    }
    const int w = (int)((cptr[(I >> 6) + 1] - cptr[I >> 6]) >> 6);
    for (int k = nd + lane; k < w; k += 64) {
        ccol[base + (int64_t)k * 64] = I;
        cval[base + (int64_t)k * 64] = 0.0;
    }
}

// Coarse rows that the hashed kernel above could not take (more than
// kGalCand candidates or kGalDistinct distinct columns; in biglist): the
// candidates as (coarse column, fine position) keys, bitonic-sorted in LDS,
// each coarse entry summing its candidates in gather order.  mode 0:
// rowlen[I] = number of coarse columns; mode 1: write them (SELL).  More
// than CAP candidates: *overflow.
template <int CAP>
__device__ inline void galerkin_sorted_row(uint64_t *key, const Sell<double> &A, const int32_t *__restrict__ Jcol,
                                           const double *__restrict__ apv, const int32_t *__restrict__ apn,
                                           const int32_t *__restrict__ mptr, const int32_t *__restrict__ mrows,
                                           int32_t I, int mode, int32_t *__restrict__ rowlen,
                                           const int64_t *__restrict__ cptr, int32_t *__restrict__ ccol,
                                           double *__restrict__ cval, int *__restrict__ overflow) {
    const int lane = threadIdx.x;
    int m = 0;
    bool over = false;
    const int32_t t1 = mptr[I + 1];
    for (int32_t t0 = mptr[I]; t0 < t1; t0 += 64) {
        const int32_t t = t0 + lane;
        int c = 0;
        int64_t b = 0;
        if (t < t1) {
            const int32_t r = mrows[t];
            b = A.ptr[r >> 6] + (r & 63);
            c = apn[r];
        }
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        const int tot = __shfl(incl, 63, 64);
        if (m + tot > CAP) {
            over = true;
            break;
        }
        const int off = m + incl - c;
        for (int k = 0; k < c; ++k) {
            const int64_t q = b + (int64_t)k * 64;
            key[off + k] = ((uint64_t)(uint32_t)Jcol[q] << 32) | (uint64_t)(uint32_t)q;
        }
        m += tot;
    }
    if (over) {
        if (lane == 0) {
            atomicOr(overflow, 1);
            if (mode == 0) rowlen[I] = 1;
        }
        return;
    }
    int mp = 1;
    while (mp < m) mp <<= 1;
    for (int k = m + lane; k < mp; k += 64) key[k] = ~0ull;
    __syncthreads();
    for (int k = 2; k <= mp; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = lane; i < mp; i += 64) {
                const int p = i ^ j;
                if (p > i) {
                    const uint64_t a = key[i], b = key[p];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) {
                        key[i] = b;
                        key[p] = a;
                    }
                }
            }
            __syncthreads();
        }
    const int C = mp / 64 > 0 ? mp / 64 : 1;
    const int lo = min(m, lane * C), hi = min(m, lo + C);
    int nh = 0;
    for (int t = lo; t < hi; ++t) nh += (t == 0 || (key[t] >> 32) != (key[t - 1] >> 32));
    int incl = nh;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    const int total = __shfl(incl, 63, 64);
    if (mode == 0) {
        if (lane == 0) rowlen[I] = total;
        return;
    }
    int rank = incl - nh;
    const int64_t base = cptr[I >> 6] + (I & 63);
    for (int t = lo; t < hi; ++t) {
        if (!(t == 0 || (key[t] >> 32) != (key[t - 1] >> 32))) continue;
        const uint32_t J = (uint32_t)(key[t] >> 32);
        double s = 0.0;
        for (int u = t; u < m && (uint32_t)(key[u] >> 32) == J; ++u) s += apv[(uint32_t)key[u]];
        ccol[base + (int64_t)rank * 64] = (int32_t)J;
        cval[base + (int64_t)rank * 64] = s;
        ++rank;
    }
    const int w = (int)((cptr[(I >> 6) + 1] - cptr[I >> 6]) >> 6);
    for (int k = total + lane; k < w; k += 64) {
        ccol[base + (int64_t)k * 64] = I;
        cval[base + (int64_t)k * 64] = 0.0;
    }
}
template <int CAP>
__global__ __launch_bounds__(64) void galerkin_kernel(Sell<double> A, const int32_t *__restrict__ Jcol,
                                                      const double *__restrict__ apv, const int32_t *__restrict__ apn,
                                                      const int32_t *__restrict__ mptr, const int32_t *__restrict__ mrows,
                                                      int mode, const int32_t *__restrict__ biglist,
                                                      const int *__restrict__ nbig, int32_t *__restrict__ rowlen,
                                                      const int64_t *__restrict__ cptr, int32_t *__restrict__ ccol,
                                                      double *__restrict__ cval, int *__restrict__ overflow) {
    __shared__ uint64_t key[CAP];
    for (int it = blockIdx.x; it < *nbig; it += gridDim.x) {
        galerkin_sorted_row<CAP>(key, A, Jcol, apv, apn, mptr, mrows, biglist[it], mode, rowlen, cptr, ccol, cval,
                                 overflow);
        __syncthreads();
    }
}

// slice widths (max row length of each 64-row slice)
__global__ __launch_bounds__(64) void slice_width_kernel(int32_t n, const int32_t *__restrict__ rowlen,
                                                         int32_t *__restrict__ width, int32_t *__restrict__ cnt) {
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    int c = i < n ? rowlen[i] : 0;
    int t = c;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c = max(c, __shfl_down(c, o, 64));
        t += __shfl_down(t, o, 64);
    }
    if (threadIdx.x == 0) {
        width[blockIdx.x] = c;
        cnt[blockIdx.x] = t;
    }
}
// rows beyond n in the last slice: padding pointing at row 0
__global__ __launch_bounds__(64) void slice_tail_kernel(int32_t n, const int64_t *__restrict__ ptr,
                                                        int32_t *__restrict__ col, double *__restrict__ val) {
    const int32_t sl = n >> 6;
    const int lane = threadIdx.x;
    if ((n & 63) == 0 || lane < (n & 63)) return;
    for (int64_t q = ptr[sl] + lane; q < ptr[sl + 1]; q += 64) {
        col[q] = 0;
        val[q] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// coarsest level: dense inverse
// ---------------------------------------------------------------------------
// What a block step of the inversion reads beside its own tile: the pivot rows
// R (kGJ x n) and the pivot columns U (n x kGJ) of M, apart from M, which the
// step writes in place.
struct GjPanels {
    double *U, *R;
};
// D = A, dense row-major, one wavefront per row, and the first panels.  A row's
// entries have distinct columns (padding entries are zero).
constexpr int kDenseMax = 1024;
constexpr int kGJ = 64;
__global__ __launch_bounds__(64) void dense_from_sell_kernel(Sell<double> A, double *__restrict__ D, GjPanels P) {
    __shared__ double row[kDenseMax];
    const int32_t n = A.n, i = blockIdx.x;
    const int lane = threadIdx.x;
    for (int j = lane; j < n; j += 64) row[j] = 0.0;
    __syncthreads();
    const int64_t b0 = A.ptr[i >> 6] + (i & 63), w = (A.ptr[(i >> 6) + 1] - A.ptr[i >> 6]) >> 6;
    for (int64_t k = lane; k < w; k += 64) {
        const double v = A.val[b0 + 64 * k];
        if (v != 0.0) row[A.col[b0 + 64 * k]] = v;
    }
    __syncthreads();
    for (int j = lane; j < n; j += 64) {
        D[(int64_t)i * n + j] = row[j];
        if (i < kGJ) P.R[(int64_t)i * n + j] = row[j];
    }
    if (lane < n) P.U[(int64_t)i * kGJ + lane] = row[lane];
}
// Blocked Gauss-Jordan inversion of an SPD matrix (no pivoting needed: every
// pivot block is a Schur complement of an SPD matrix, hence SPD).  With P the
// next kGJ indices, R the others and B = M[P,P]^-1 the block step is
//   V = B M[P,R],  W = M[R,P] B,
//   M[R,R] = M[R,R] - M[R,P] V,  M[P,R] = V,  M[R,P] = -W,  M[P,P] = B,
// one launch, one workgroup per 64 x 64 tile: each tile of M[R,R] forms its own
// tile of V, and the workgroup of the next pivot block inverts it before it
// ends.  A workgroup reads its own tile of M and otherwise the panels, of which
// it also writes its share for the next step (from one copy of M to another the
// same bits took as long and 8 MB more at 1000 rows).  That inversion is the chain that the
// steps wait for (~20 us); the products, loads and launches around it were 33
// us of a step as four kernels (pivot, panels, update, write-back in place: 62
// us a step, now 27; 430 rows 434 -> 218 us).
constexpr int kGJLd = kGJ + 2;  // of a tile in LDS: rows 16 bytes aligned, their banks shifted
constexpr int kQ = 4;  // pivots eliminated together inside the diagonal block

// The inverse of the k x k block t (padded by the identity), in place.  256 threads as a 16 x 16
// grid, each keeping a 4 x 4 tile of the (identity-padded) 64 x 64 block in
// registers.  The elimination takes kQ pivots per step: the owners publish
// the kQ pivot rows and columns in LDS (double-buffered, one barrier per
// step), every thread inverts the kQ x kQ pivot block itself and updates its
// tile by the block rule above, restricted to the diagonal block.
__device__ inline void inv4(double b[kQ][kQ]) {
#pragma unroll
    for (int p = 0; p < kQ; ++p) {
        const double pinv = 1.0 / b[p][p];
        double pr[kQ];  // the pivot row before this step
#pragma unroll
        for (int j = 0; j < kQ; ++j) pr[j] = b[p][j];
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const double ca = b[i][p] * pinv;
#pragma unroll
            for (int j = 0; j < kQ; ++j)
                b[i][j] = (i == p) ? (j == p ? pinv : pr[j] * pinv) : (j == p ? -ca : b[i][j] - ca * pr[j]);
        }
    }
}
__device__ inline void gj_invert(double (&t)[4][4], int k) {
    __shared__ double rowp[2][kQ][kGJ], colp[2][kGJ][kQ];
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    const int nsteps = (k + kQ - 1) / kQ;
    for (int pb = 0; pb < nsteps; ++pb) {
        const int buf = pb & 1;
        const bool ip = ty == pb, jp = tx == pb;
        if (ty == pb) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) rowp[buf][a][tx * 4 + c] = t[a][c];
        }
        if (tx == pb) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) colp[buf][ty * 4 + a][c] = t[a][c];
        }
        __syncthreads();
        double B[kQ][kQ], C[4][kQ], R[kQ][4];
#pragma unroll
        for (int a = 0; a < kQ; ++a)
#pragma unroll
            for (int c = 0; c < kQ; ++c) B[a][c] = rowp[buf][a][pb * 4 + c];
        inv4(B);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < kQ; ++c) C[a][c] = colp[buf][ty * 4 + a][c];
#pragma unroll
        for (int a = 0; a < kQ; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) R[a][c] = rowp[buf][a][tx * 4 + c];
        // CB = C B (rows of the tile against the pivot block)
        double CB[4][kQ];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < kQ; ++c) {
                double v = 0.0;
#pragma unroll
                for (int m = 0; m < kQ; ++m) v += C[a][m] * B[m][c];
                CB[a][c] = v;
            }
        #pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // the pivot rows' block B R, or what is left of t
                double x = ip ? 0.0 : t[a][c];
#pragma unroll
                for (int m = 0; m < kQ; ++m) x = fma(ip ? B[a][m] : -CB[a][m], R[m][c], x);
                t[a][c] = jp ? (ip ? B[a][c] : -CB[a][c]) : x;
            }
    }
}
// Stores the inverse (zeros past k) where the next step reads it.
__device__ inline void gj_put(const double (&t)[4][4], int k, double *__restrict__ B) {
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = ty * 4 + a, j = tx * 4 + c;
            B[i * kGJ + j] = i < k && j < k ? t[a][c] : 0.0;
        }
}
__global__ __launch_bounds__(256) void gj_first_kernel(int32_t n, const double *__restrict__ M,
                                                       double *__restrict__ B) {
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15, k = min(n, kGJ);
    double t[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = ty * 4 + a, j = tx * 4 + c;
            // every lane loads (the padding from the block's first entry) so the
            // sixteen loads are in flight together
            const bool in = i < k && j < k;
            const double x = M[in ? (int64_t)i * n + j : 0];
            t[a][c] = in ? x : (i == j ? 1.0 : 0.0);
        }
    gj_invert(t, k);
    gj_put(t, k, B);
}

// acc = A B over k: thread (ty, tx) the rows 4 ty + a and columns 4 tx + c,
// every entry a chain over m in order
__device__ inline void gj_product(const double (&A)[kGJ][kGJLd], const double (&B)[kGJ][kGJLd], int k,
                                  double (&acc)[4][4]) {
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = 0.0;
#pragma unroll 2
    for (int m = 0; m < k; m += 2) {  // the tiles are zero past k
        double2 x[4], y[2][2];
#pragma unroll
        for (int a = 0; a < 4; ++a) x[a] = *reinterpret_cast<const double2 *>(&A[ty * 4 + a][m]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) y[u][h] = *reinterpret_cast<const double2 *>(&B[m + u][tx * 4 + 2 * h]);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                acc[a][2 * h] = fma(x[a].y, y[1][h].x, fma(x[a].x, y[0][h].x, acc[a][2 * h]));
                acc[a][2 * h + 1] = fma(x[a].y, y[1][h].y, fma(x[a].x, y[0][h].y, acc[a][2 * h + 1]));
            }
    }
}
// One block step with pivots [p0, p0 + k) on M, given its panels and B =
// M[P,P]^-1; the panels and next = the inverse of the following pivot block.
__global__ __launch_bounds__(256) void gj_step_kernel(int32_t n, int32_t p0, int32_t k,
                                                      double *__restrict__ M, GjPanels P, GjPanels Pnext,
                                                      const double *__restrict__ B, double *__restrict__ next) {
    __shared__ __align__(16) double S[kGJ][kGJLd], T[kGJ][kGJLd];
    const int32_t i0 = blockIdx.y * kGJ, j0 = blockIdx.x * kGJ;
    const bool ri = i0 == p0, rj = j0 == p0;
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    constexpr int kIt = kGJ * kGJ / 256;
    // S and T: B and M[P,J], or for the column panel M[I,P] and B.  Clamped
    // addresses and selects rather than conditional loads, so that all loads
    // are issued before the first wait.
    double u[kIt];  // M[I,P]: S for the column panel, the second product's S for M[R,R]
    double v[kIt];  // M[P,J]
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int e = threadIdx.x + it * 256, r = e >> 6, c = e & 63;
        const bool iu = i0 + r < n && c < k, iv = r < k && j0 + c < n;
        const double b = B[e];
        const double x = P.U[(int64_t)(iu ? i0 + r : 0) * kGJ + (iu ? c : 0)];
        const double y = P.R[(int64_t)(iv ? r : 0) * n + (iv ? j0 + c : 0)];
        u[it] = iu ? x : 0.0;
        v[it] = iv ? y : 0.0;
        S[r][c] = rj && !ri ? u[it] : b;
        T[r][c] = rj ? b : v[it];
    }
    __syncthreads();
    double out[4][4];
    if (ri && rj) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) out[a][c] = S[ty * 4 + a][tx * 4 + c];
    } else {
        double acc[4][4];
        gj_product(S, T, k, acc);
        if (rj) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) out[a][c] = -acc[a][c];
        } else if (ri) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) out[a][c] = acc[a][c];
        } else {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int i = i0 + ty * 4 + a, j = j0 + tx * 4 + c;
                    const bool in = i < n && j < n;
                    out[a][c] = M[in ? (int64_t)i * n + j : (int64_t)i0 * n + j0];  // of its own tile
                }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < kIt; ++it) {
                const int e = threadIdx.x + it * 256;
                S[e >> 6][e & 63] = u[it];
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) T[ty * 4 + a][tx * 4 + c] = acc[a][c];
            __syncthreads();
            gj_product(S, T, k, acc);
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) out[a][c] -= acc[a][c];
        }
    }
    if (i0 == j0 && i0 == p0 + kGJ) {  // the next pivot block
        const int kn = min(kGJ, n - i0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = ty * 4 + a, j = tx * 4 + c;
                if (i >= kn || j >= kn) out[a][c] = i == j ? 1.0 : 0.0;
            }
        gj_invert(out, kn);
        gj_put(out, kn, next);
        return;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = i0 + ty * 4 + a, j = j0 + tx * 4 + c;
            if (i < n && j < n) {
                M[(int64_t)i * n + j] = out[a][c];
                if (j0 == p0 + kGJ) Pnext.U[(int64_t)i * kGJ + j - j0] = out[a][c];
                if (i0 == p0 + kGJ) Pnext.R[(int64_t)(i - i0) * n + j] = out[a][c];
            }
        }
}

// ---------------------------------------------------------------------------
// V-cycle kernels
// ---------------------------------------------------------------------------
// x = M^-1 b (first sweep from zero)
template <class X>
__global__ __launch_bounds__(kAT) void vc_scale_kernel(int32_t n, const X *__restrict__ dinv, const X *__restrict__ b,
                                                       X *__restrict__ x, const PcgState *st) {
    if (st && st->done) return;
    GS(i, n) x[i] = dinv[i] * b[i];
}
// r = b - A x
template <class V, class X>
__global__ __launch_bounds__(kAT) void vc_resid_kernel(Sell<V> A, const X *__restrict__ b, const X *__restrict__ x,
                                                       X *__restrict__ r, const PcgState *st) {
    if (st && st->done) return;
    GS(i, A.n) r[i] = b[i] - sell_row_apply<V, X>(A, (int32_t)i, [&](int32_t j) { return x[j]; });
}
// b_c[I] = sum of r over aggregate I: kRL lanes per coarse row (four coarse
// rows per wavefront), members strided over the lanes and combined by a fixed
// shuffle tree.  With xc, also the first smoothing iterate of the coarse
// level, xc = D_c^-1 bc.
constexpr int kRL = 16;
template <class X>
__global__ __launch_bounds__(kAT) void vc_restrict_kernel(int32_t nc, const int32_t *__restrict__ mptr,
                                                          const int32_t *__restrict__ mrows, const X *__restrict__ r,
                                                          X *__restrict__ bc, const X *__restrict__ dinv_c,
                                                          X *__restrict__ xc, const PcgState *st) {
    if (st && st->done) return;
    const int sub = threadIdx.x & (kRL - 1);
    const int64_t g0 = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) / kRL;
    const int64_t ng = ((int64_t)gridDim.x * blockDim.x) / kRL;
    // every lane of a wavefront runs the same number of passes (the shuffles need them all)
    for (int64_t gb = g0 - (g0 & (64 / kRL - 1)); gb < nc; gb += ng) {
        const int64_t I = gb + (g0 & (64 / kRL - 1));
        X s = 0;
        if (I < nc)
            for (int32_t t = mptr[I] + sub; t < mptr[I + 1]; t += kRL) s += r[mrows[t]];
#pragma unroll
        for (int o = kRL / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (sub == 0 && I < nc) {
            bc[I] = s;
            if (xc) xc[I] = dinv_c[I] * s;
        }
    }
}
// y = x + P e (injection from the aggregate)
template <class X>
__global__ __launch_bounds__(kAT) void vc_prolong_kernel(int32_t n, const X *__restrict__ x,
                                                         const int32_t *__restrict__ agg, const X *__restrict__ e,
                                                         X *__restrict__ y, const PcgState *st) {
    if (st && st->done) return;
    GS(i, n) y[i] = x[i] + e[agg[i]];
}
// out = y + M^-1 (b - A y); with rz, also the block partials of b . out (the
// CG scalar r.z when this is the last sweep of a V-cycle on level 0)
// With zq also the partials of qv . out (flexible CG: the new preconditioned
// residual against the last A p).
template <class V, class X>
__global__ __launch_bounds__(kAT) void vc_sweep_kernel(Sell<V> A, const X *__restrict__ dinv, const X *__restrict__ b,
                                                       const X *__restrict__ y, X *__restrict__ out,
                                                       const PcgState *st) {
    if (st && st->done) return;
    GS(i, A.n) {
        const X s = sell_row_apply<V, X>(A, (int32_t)i, [&](int32_t j) { return y[j]; });
        out[i] = y[i] + dinv[i] * (b[i] - s);
    }
}
// (levels of more than kSplitMaxRows rows)
template <class V, class X>
__global__ __launch_bounds__(kKrylovThreads) void vc_sweep_rz_kernel(Sell<V> A, const X *__restrict__ dinv,
                                                                     const X *__restrict__ b, const X *__restrict__ y,
                                                                     X *__restrict__ out, double *__restrict__ rz,
                                                                     double *__restrict__ zq,
                                                                     const X *__restrict__ qv, const PcgState *st) {
    if (st && st->done) return;
    double v[2] = {0.0, 0.0};
    for (int64_t i = (int64_t)xcd_block() * kKrylovThreads + threadIdx.x; i < A.n;
         i += (int64_t)gridDim.x * kKrylovThreads) {
        const X yi = y[i], di = dinv[i], bi = b[i];  // ahead of the row, not a second wait after it
        const X s = sell_row_apply<V, X>(A, (int32_t)i, [&](int32_t j) { return y[j]; });
        const X o = yi + di * (bi - s);
        out[i] = o;
        v[0] += (double)bi * (double)o;
        if (zq) v[1] += (double)qv[i] * (double)o;
    }
    block_reduce<OpSum, 2, kKrylovThreads>(v);
    if (threadIdx.x == 0) {
        rz[blockIdx.x] = v[0];
        if (zq) zq[blockIdx.x] = v[1];
    }
}
// prolongation and sweep in one pass (small levels): y = x + P e with
// x = D^-1 b formed on the fly, out = y + D^-1 (b - A y)
template <class V, class X>
__global__ __launch_bounds__(kAT) void vc_post_fused_kernel(Sell<V> A, const X *__restrict__ dinv,
                                                            const X *__restrict__ b, const int32_t *__restrict__ agg,
                                                            const X *__restrict__ e, X *__restrict__ out,
                                                            const PcgState *st) {
    if (st && st->done) return;
    GS(i, A.n) {
        const X s = sell_row_apply<V, X>(A, (int32_t)i, [&](int32_t j) { return dinv[j] * b[j] + e[agg[j]]; });
        const X yi = dinv[i] * b[i] + e[agg[i]];
        out[i] = yi + dinv[i] * (b[i] - s);
    }
}
// Small levels (at most kSmallRows rows): kG lanes per row, lane g taking the
// row's slots g, g + kG, ..., the kG partial sums combined by a fixed
// butterfly, so a row's gathers are spread over several lanes and fewer
// dependent loads sit on one lane.  The lanes of one slot index read
// consecutive rows (coalesced).  MODE 0: out = b - A x.  MODE 1: out = x +
// D^-1 (b - A x).  MODE 2: with y = D^-1 b + P e, out = y + D^-1 (b - A y).
// MODE 3: with y = x + P e, out = y + D^-1 (b - A y).
constexpr int kG = 4;
constexpr int kRowsPerWave = 64 / kG;
template <int MODE, class V, class X>
__global__ __launch_bounds__(kAT) void vc_small_kernel(Sell<V> A, const X *__restrict__ dinv,
                                                       const X *__restrict__ b, const X *__restrict__ x,
                                                       const int32_t *__restrict__ agg, const X *__restrict__ e,
                                                       X *__restrict__ out, const PcgState *st) {
    if (st && st->done) return;
    const int lane = threadIdx.x & 63;
    const int g = lane / kRowsPerWave, rr = lane % kRowsPerWave;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    auto f = [&](int32_t j) -> X {
        if constexpr (MODE <= 1) return x[j];
        else if constexpr (MODE == 2) return dinv[j] * b[j] + e[agg[j]];
        else return x[j] + e[agg[j]];
    };
    for (int64_t w = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) >> 6; w * kRowsPerWave < A.n; w += nw) {
        const int32_t i = (int32_t)(w * kRowsPerWave) + rr;
        const X sum = lane_row(A, i, f).template sum<X, 2>([](X t) { return t; });
        if (g == 0 && i < A.n) {
            if constexpr (MODE == 0) {
                out[i] = b[i] - sum;
            } else {
                X yi;
                if constexpr (MODE == 1) yi = x[i];
                else if constexpr (MODE == 2) yi = dinv[i] * b[i] + e[agg[i]];
                else yi = x[i] + e[agg[i]];
                out[i] = yi + dinv[i] * (b[i] - sum);
            }
        }
    }
}
static inline unsigned grid_small(int32_t n) {
    return (unsigned)std::max<int64_t>(1, ((int64_t)n * kG + kAT - 1) / kAT);
}

// ---------------------------------------------------------------------------
// K-cycle: on a coarse level m the coarse correction is two steps of a
// flexible CG on A_m e = b, each preconditioned by the V-cycle from level m
// (Krylov acceleration of the coarse-grid correction, which unsmoothed
// aggregation needs to keep its convergence independent of the level count).
// With c = B(b), v = A c, rho = c.v, alpha1 = c.b / rho, rt = b - alpha1 v,
// d = B(rt), w = A d, gamma = d.v, beta = d.w - gamma^2 / rho,
// alpha2 = d.rt / beta:   e = (alpha1 - gamma alpha2 / rho) c + alpha2 d.
// Scalars are formed by each consuming kernel from per-block partials, in a
// fixed order.  parts: [c.v | c.b | d.w | d.v | d.rt] x G.
// ---------------------------------------------------------------------------
// Up to kSmallRows rows the partials are sums of 64-row slices (4 per 256 rows,
// zeros past the last), from kernels with 4 lanes per row; above, one per block
// of 256 threads that strides over the rows (kReduceBlocks of them).  Summed
// here in the order of the latter, whichever kernels wrote them.
template <int NT, int NV, class P>
__device__ inline void kc_sums(bool slices, P p, int G, double (&v)[NV]) {
    static_assert(NT >= 256, "one thread per group of partials");
    __shared__ double lds[NV][4];
    const int t = threadIdx.x;
    if (t < 256) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const double *q = p(k);
            double s = 0.0;
            if (slices) {
                for (int g = 4 * t; g < G; g += 1024) s += ((q[g] + q[g + 1]) + q[g + 2]) + q[g + 3];
            } else {
                for (int g = t; g < G; g += 256) s += q[g];
            }
            s = wave_reduce<OpSum>(s);
            if ((t & 63) == 0) lds[k][t >> 6] = s;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = lds[k][0];
        for (int w = 1; w < 4; ++w) v[k] += lds[k][w];
    }
    __syncthreads();
}
struct KcParts {
    double *base;
    int G;
    bool slices;
    __device__ double *at(int k) const { return base + (size_t)k * G; }
};
template <int NT>
__device__ inline double kc_alpha1(const KcParts &P) {
    double t[2];
    kc_sums<NT>(P.slices, [&](int k) { return P.at(k); }, P.G, t);
    return t[0] > 0.0 ? t[1] / t[0] : 0.0;
}
// the correction a level takes from the one below: e, or with d the K-cycle's
// combination ac e + ad d
template <class X>
struct KcE {
    const X *e, *d;
    KcParts P;
};
template <int NT, class X>
__device__ inline void kc_weights(const KcE<X> &E, X &ac, X &ad) {
    ac = 1;
    ad = 0;
    if (!E.d) return;  // uniform
    double t[5];
    kc_sums<NT>(E.P.slices, [&](int k) { return E.P.at(k); }, E.P.G, t);
    const double rho = t[0];
    double a1 = 0.0, g = 0.0, a2 = 0.0;
    if (rho > 0.0) {
        a1 = t[1] / rho;
        g = t[3];
        const double beta = t[2] - g * g / rho;
        a2 = beta > 0.0 ? t[4] / beta : 0.0;
    }
    ac = (X)(rho > 0.0 ? a1 - g * a2 / rho : 0.0);
    ad = (X)a2;
}
template <class X>
__device__ inline X kc_e(X ac, X ad, X e, X d) {
    return fma(ac, e, ad * d);
}
// v = A c; partials c.v and c.b
template <bool SPLIT, class V, class X>
__global__ __launch_bounds__(kAT) void kc_av_kernel(Sell<V> A, const X *__restrict__ c, const X *__restrict__ b,
                                                    X *__restrict__ v, KcParts P, const PcgState *st) {
    if (st && st->done) return;
    auto f = [&](int32_t j) { return c[j]; };
    auto row = [&](int32_t i, X vi, double *p) {
        v[i] = vi;
        p[0] += (double)c[i] * (double)vi;
        p[1] += (double)c[i] * (double)b[i];
    };
    auto put = [&](int k) { return P.at(k); };
    if constexpr (SPLIT) {
        const int32_t i = split_row<kAT, false>();
        const X s = lane_row(A, i, f).template sum<X, 1>([](X t) { return t; });
        split_rows<kAT, 2, false>(A.n, P.G, i, s, row, put);
    } else {
        krylov_rows<kAT, 2, false, V, X>(A, false, P.G, f, row, put);
    }
}
// rt = b - alpha1 v, and the next V-cycle's first iterate xa = D^-1 rt
template <class X>
__global__ __launch_bounds__(kAT) void kc_rt_kernel(int32_t n, const X *__restrict__ b, const X *__restrict__ v,
                                                    const X *__restrict__ dinv, KcParts P, X *__restrict__ rt,
                                                    X *__restrict__ xa, const PcgState *st) {
    if (st && st->done) return;
    const X a = (X)kc_alpha1<kAT>(P);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const X r = b[i] - a * v[i];
        rt[i] = r;
        xa[i] = dinv[i] * r;
    }
}
// The same (xa is not needed) with the next V-cycle's residual r = rt - A D^-1 rt,
// in one launch: levels of at most kSmallRows rows, where a launch (~3 us of the
// host's time) costs more than forming rt again at every gathered entry.
template <class V, class X>
__global__ __launch_bounds__(kAT) void kc_rt_resid_kernel(Sell<V> A, const X *__restrict__ b, const X *__restrict__ v,
                                                          const X *__restrict__ dinv, KcParts P, X *__restrict__ rt,
                                                          X *__restrict__ r, const PcgState *st) {
    if (st && st->done) return;
    const int lane = threadIdx.x & 63;
    const int32_t i = (int32_t)(((int64_t)xcd_block() * kAT + threadIdx.x) >> 6) * kSplitRows + lane % kSplitRows;
    struct Raw {
        X b, v, d;
    };
    auto R = lane_row(A, i, [&](int32_t j) { return Raw{b[j], v[j], dinv[j]}; });
    const X a = (X)kc_alpha1<kAT>(P);
    const X s = R.template sum<X, 2>([&](const Raw &w) {
        const X t = w.b - a * w.v;
        return w.d * t;
    });
    if (lane < kSplitRows && i < A.n) {
        const X t = b[i] - a * v[i];
        rt[i] = t;
        r[i] = t - s;
    }
}
// partials d.w (w = A d), d.v, d.rt
template <bool SPLIT, class V, class X>
__global__ __launch_bounds__(kAT) void kc_aw_kernel(Sell<V> A, const X *__restrict__ d, const X *__restrict__ v,
                                                    const X *__restrict__ rt, KcParts P, const PcgState *st) {
    if (st && st->done) return;
    auto f = [&](int32_t j) { return d[j]; };
    auto row = [&](int32_t i, X wi, double *p) {
        p[0] += (double)d[i] * (double)wi;
        p[1] += (double)d[i] * (double)v[i];
        p[2] += (double)d[i] * (double)rt[i];
    };
    auto put = [&](int k) { return P.at(2 + k); };
    if constexpr (SPLIT) {
        const int32_t i = split_row<kAT, false>();
        const X s = lane_row(A, i, f).template sum<X, 1>([](X t) { return t; });
        split_rows<kAT, 3, false>(A.n, P.G, i, s, row, put);
    } else {
        krylov_rows<kAT, 3, false, V, X>(A, false, P.G, f, row, put);
    }
}
// e = (alpha1 - gamma alpha2 / rho) c + alpha2 d
template <class X>
__global__ __launch_bounds__(kAT) void kc_combine_kernel(int32_t n, KcE<X> E, X *__restrict__ e, const PcgState *st) {
    if (st && st->done) return;
    X ac, ad;
    kc_weights<kAT>(E, ac, ad);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        e[i] = kc_e(ac, ad, E.e[i], E.d[i]);
}

// ---------------------------------------------------------------------------
// CG around a finest level of at most kSplitMaxRows rows: fewer launches.
// There an iteration is bound by its launches and by each kernel's one chain of
// loads.  Five kernels and 26 us of them per two-level iteration at 1089 rows
// (product, residual and sweep alone were 10 us each); a time step on 10^3
// cells with its set-up 441 -> 330 launches, 2540 -> 1980 us; on 33x37x35 cells
// 5040 -> 4380 us
// ---------------------------------------------------------------------------
// CG's update and the V-cycle's first residual: x += alpha p, r_out = r_in -
// alpha q, x0 = D^-1 r_out, res = r_out - A x0 (x0 formed again at every
// gathered entry), partials of r_out . r_out
template <class V>
__global__ __launch_bounds__(kSplitThreads) void pcg_update_resid_kernel(
    Sell<V> A, int k, double *__restrict__ x, const double *__restrict__ r_in, double *__restrict__ r_out,
    const double *__restrict__ p, const double *__restrict__ q, const double *__restrict__ dinv,
    double *__restrict__ x0, double *__restrict__ res, PcgParts P, PcgState *st) {
    if (st->done) return;
    const int32_t i = split_row<kSplitThreads, false>();
    struct Raw {
        double r, q, d;
    };
    auto R = lane_row(A, i, [&](int32_t j) { return Raw{r_in[j], q[j], dinv[j]}; });
    double t[2];
    krylov_sums<kSplitThreads>(true, [&](int m) { return m ? P.pq(k) : P.rz(k - 1); }, P.G, t);
    const double a = t[0] / t[1];
    const double s = R.template sum<double, 2>([&](const Raw &w) {
        const double rj = w.r - a * w.q;
        return w.d * rj;
    });
    split_rows<kSplitThreads, 1, false>(
        A.n, P.G, i, s,
        [&](int32_t m, double sm, double *v) {
            x[m] += a * p[m];
            const double ri = r_in[m] - a * q[m];
            r_out[m] = ri;
            x0[m] = dinv[m] * ri;
            res[m] = ri - sm;
            v[0] += ri * ri;
        },
        [&](int) { return P.rr(k); });
    if (threadIdx.x == 0 && blockIdx.x == 0) st->iter = k + 1;
}
// the prolongation and the last sweep: out = y + D^-1 (b - A y) with y = x + P e,
// partials of b . out and (with zq) qv . out
template <class V, class X>
__global__ __launch_bounds__(kSplitThreads) void vc_post_rz_kernel(
    Sell<V> A, int G, const X *__restrict__ dinv, const X *__restrict__ b, const X *__restrict__ x,
    const int32_t *__restrict__ agg, KcE<X> E, X *__restrict__ out, double *__restrict__ rz, double *__restrict__ zq,
    const X *__restrict__ qv, const PcgState *st) {
    if (st && st->done) return;
    const int32_t i = split_row<kSplitThreads, true>();
    const bool two = E.d != nullptr;
    struct Raw {
        X x, c, d;
    };
    auto R = lane_row(A, i, [&](int32_t j) {
        const int32_t J = agg[j];
        return Raw{x[j], E.e[J], two ? E.d[J] : (X)0};
    });
    X ac, ad;
    kc_weights<kSplitThreads>(E, ac, ad);
    auto use = [&](const Raw &w) -> X {
        const X e = two ? kc_e(ac, ad, w.c, w.d) : w.c;
        return w.x + e;
    };
    const X s = R.template sum<X, 1>(use);
    split_rows<kSplitThreads, 2, true>(
        A.n, G, i, s,
        [&](int32_t m, X sm, double *v) {
            const X y = use(R.gather(m));
            const X o = y + dinv[m] * (b[m] - sm);
            out[m] = o;
            v[0] += (double)b[m] * (double)o;
            if (zq) v[1] += (double)qv[m] * (double)o;
        },
        [&](int k) { return k ? zq : rz; });
}

// dense coarse solve x = Ainv b: one wavefront per row, lanes along the
// (contiguous) row, fixed-order wave reduction
template <class X>
__global__ __launch_bounds__(kAT) void vc_dense_kernel(int32_t n, const X *__restrict__ Ainv, const X *__restrict__ b,
                                                       X *__restrict__ x, const PcgState *st) {
    if (st && st->done) return;
    const int lane = threadIdx.x & 63;
    for (int64_t i = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) >> 6; i < n;
         i += ((int64_t)gridDim.x * blockDim.x) >> 6) {
        double s = 0.0;
        for (int32_t j = lane; j < n; j += 64) s += (double)Ainv[i * n + j] * (double)b[j];
        s = wave_reduce<OpSum>(s);
        if (lane == 0) x[i] = (X)s;
    }
}
// conversions for the single-precision hierarchy
__global__ __launch_bounds__(kAT) void to_float_kernel(int64_t n, const double *__restrict__ a, float *__restrict__ b) {
    GS(i, n) b[i] = (float)a[i];
}
// FP32 copy of a level's matrix that keeps every row sum: the off-diagonal
// entries are rounded to FP32 and the diagonal, kept apart in FP64, absorbs
// their rounding (dg_i = sum_j a_ij - sum_{j != i} fl32(a_ij)).  The rounding
// error is then a Laplacian-like matrix with zero row sums: it leaves the
// constant vector alone and perturbs each coupling by a relative 2^-24, so
// the near-null (smooth) modes that the coarse levels must resolve are kept.
__global__ __launch_bounds__(kAT) void to_float_rowsum_kernel(Sell<double> A, float *__restrict__ v32,
                                                              double *__restrict__ dg) {
    GS(i, A.n) {
        const int64_t b0 = A.ptr[i >> 6], b1 = A.ptr[(i >> 6) + 1];
        double s = 0.0, so = 0.0;
        for (int64_t q = b0 + (i & 63); q < b1; q += 64) {
            const double a = A.val[q];
            s += a;
            if (A.col[q] == i) {
                v32[q] = 0.0f;
            } else {
                const float f = (float)a;
                v32[q] = f;
                so += (double)f;
            }
        }
        dg[i] = s - so;
    }
}
__global__ __launch_bounds__(kAT) void to_double_kernel(int64_t n, const float *__restrict__ a, double *__restrict__ b) {
    GS(i, n) b[i] = (double)a[i];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define ALAUNCH(kern, grid, block, ...)                                              \
    do {                                                                             \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, s, __VA_ARGS__);        \
        VAG_HIP(hipGetLastError());                                                  \
    } while (0)

void amg_launch_diag(hipStream_t s, Sell<double> A, double *diag, double *dinv) {
    if (A.n > 0) ALAUNCH(amg_diag_kernel, gridv(A.n), kAT, A, diag, dinv);
}
void amg_launch_mis(hipStream_t s, Sell<double> A, const double *diag, double theta, int rounds, int hops,
                    const CoarsenInit &I, int32_t *flag, int32_t *scol, int *progress) {
    volatile int *started = progress;
    *started = 0;
    ALAUNCH(strength_kernel, gridv((int64_t)A.n + 1), kAT, A, diag, theta, scol, I);
    for (int r = 0; r < rounds; ++r) {
        int *cur = I.undecided + (int64_t)r * kCntSlots * kCntStride;
        const int *active = r ? cur - kCntSlots * kCntStride : nullptr;
        ALAUNCH(mis_max_kernel, gridv(A.n), kAT, A.n, A.ptr, scol, I.T, I.T1, active, r, progress);
        ALAUNCH(mis_select_kernel, gridv(A.n), kAT, A.n, hops, A.ptr, scol, I.T1, I.T, cur, active);
        // Stop queueing rounds once nothing is undecided.  The device says in
        // pinned memory which round it has begun; the host stays at most three
        // rounds ahead of it, so the device never waits for the host's look as
        // it did for a copy and a synchronisation every fourth round.
        poll_rounds(s, started, r - 2, kMisRounds);
        if (*started > kMisRounds) break;
    }
    ALAUNCH(mis_flag_kernel, gridv(A.n), kAT, A.n, I.T, flag);
}
static void scan_to(hipStream_t s, int32_t n, const int32_t *in, const ScanTo &to, int32_t *tmp) {
    // tmp: at least 2 * (n / 1024 + 2) ints
    const int32_t nb = (n + 256 * kScanItems - 1) / (256 * kScanItems);
    if (nb <= 8) {  // three launches cost more than eight items a thread
        ALAUNCH(scan_int_kernel, 1, 1024, n, in, to);
        return;
    }
    ALAUNCH(scan_sums_kernel, nb, 256, n, in, tmp);
    ALAUNCH(scan_int_kernel, 1, 1024, nb, tmp, (ScanTo{tmp + nb + 1, nullptr, nullptr, nullptr}));
    ALAUNCH(scan_apply_kernel, nb, 256, n, in, tmp + nb + 1, to);
}
void amg_launch_scan(hipStream_t s, int32_t n, const int32_t *in, int32_t *out, int32_t *tmp, int *host) {
    scan_to(s, n, in, ScanTo{out, nullptr, nullptr, host}, tmp);
}
void amg_launch_lonely(hipStream_t s, int32_t n, const int32_t *lonely, const int32_t *nroot, int32_t *agg,
                       int32_t *tmp, int *host) {
    scan_to(s, n, lonely, ScanTo{nullptr, agg, nroot, host}, tmp);
}
void amg_launch_aggregate(hipStream_t s, Sell<double> A, const double *diag, const int32_t *scol, const int32_t *root,
                          const int32_t *rid, int32_t *agg1, int32_t *agg, int32_t *lonely) {
    ALAUNCH(agg_pass1_kernel, gridv(A.n), kAT, A, diag, scol, root, rid, agg1);
    ALAUNCH(agg_pass2_kernel, gridv(A.n), kAT, A, diag, scol, agg1, agg, lonely);
}
void amg_launch_members(hipStream_t s, int32_t n, int32_t nc, const int32_t *agg, int32_t *cnt, int32_t *ptr,
                        int32_t *cursor, int32_t *tmp, int32_t *rows, int32_t *scan_tmp) {
    // cnt and cursor zeroed by the caller
    ALAUNCH(count_kernel, gridv(n), kAT, n, agg, cnt);
    amg_launch_scan(s, nc, cnt, ptr, scan_tmp);
    ALAUNCH(members_fill_kernel, gridv(n), kAT, n, agg, ptr, cursor, tmp);
    ALAUNCH(members_rank_kernel, reduce_grid((int64_t)nc * 64, kAT), kAT, nc, ptr, tmp, rows);
}
void amg_launch_collapse(hipStream_t s, Sell<double> A, const int32_t *agg, int32_t *apJ, double *apv,
                         int32_t *apn, int32_t *spill, int *nspill) {
    ALAUNCH(ap_collapse_kernel, gridv(A.n), kAT, A, agg, apJ, apv, apn, spill, nspill);
    ALAUNCH(ap_spill_kernel<1024>, 2048, 64, A, agg, apJ, apv, apn, spill, nspill);
}
void amg_launch_galerkin(hipStream_t s, Sell<double> A, const int32_t *Jcol, const double *apv, const int32_t *apn,
                         const int32_t *mptr, const int32_t *mrows, int32_t nc, int mode, int32_t *big,
                         int32_t *biglist, int *nbig, int32_t *rowlen, const int64_t *cptr, int32_t *ccol,
                         double *cval, int *overflow) {
    if (nc <= 0) return;
    ALAUNCH(galerkin_hash_kernel, nc, 64, A, Jcol, apv, apn, mptr, mrows, nc, mode, big, biglist, nbig, rowlen, cptr,
            ccol, cval);
    // 512 blocks: two of these keys fit on a CU, and usually there is no such row
    ALAUNCH(galerkin_kernel<8192>, std::min(nc, 512), 64, A, Jcol, apv, apn, mptr, mrows, mode, biglist, nbig, rowlen,
            cptr, ccol, cval, overflow);
}
void amg_launch_slices(hipStream_t s, int32_t n, const int32_t *rowlen, int32_t *width, int32_t *cnt, int64_t *ptr,
                       unsigned long long *nnz, int64_t *host, const int *flag, int *host_flag) {
    const int32_t ns = (n + 63) / 64;
    if (ns > 0) ALAUNCH(slice_width_kernel, ns, 64, n, rowlen, width, cnt);
    launch_slice_scan(s, ns, width, kSliceRows, ptr, cnt, nnz, host, flag, host_flag);
}
void amg_launch_slice_tail(hipStream_t s, int32_t n, const int64_t *ptr, int32_t *col, double *val) {
    if (n & 63) ALAUNCH(slice_tail_kernel, 1, 64, n, ptr, col, val);
}
void amg_launch_dense_inverse(hipStream_t s, Sell<double> A, double *D, double *work) {
    const int32_t n = A.n;
    if (n > kDenseMax) throw Error(VAG_ERR_ARG, "internal: dense inverse of too many rows");
    const int nt = (n + kGJ - 1) / kGJ;
    double *B[2] = {work, work + kGJ * kGJ};
    GjPanels P[2];
    for (int h = 0; h < 2; ++h) {
        P[h].U = work + 2 * kGJ * kGJ + (int64_t)h * 2 * kGJ * n;
        P[h].R = P[h].U + (int64_t)kGJ * n;
    }
    ALAUNCH(dense_from_sell_kernel, n, 64, A, D, P[0]);
    ALAUNCH(gj_first_kernel, 1, 256, n, D, B[0]);
    for (int p = 0; p < nt; ++p) {
        hipLaunchKernelGGL(gj_step_kernel, dim3(nt, nt), dim3(256), 0, s, n, p * kGJ, std::min(kGJ, n - p * kGJ), D,
                           P[p & 1], P[(p & 1) ^ 1], B[p & 1], B[(p & 1) ^ 1]);
        VAG_HIP(hipGetLastError());
    }
}
int kc_grid(int32_t n) {
    const int b = (int)reduce_grid(n, kAT);
    return n <= kSmallRows ? 4 * b : b;
}
static inline KcParts kc_parts(double *base, int32_t n) { return KcParts{base, kc_grid(n), n <= kSmallRows}; }
template <class V, class X>
void amg_launch_kc_av(hipStream_t s, Sell<V> A, const X *c, const X *b, X *v, double *parts, const PcgState *st) {
    if (A.n <= kSmallRows)
        ALAUNCH((kc_av_kernel<true, V, X>), kc_grid(A.n), kAT, A, c, b, v, kc_parts(parts, A.n), st);
    else
        ALAUNCH((kc_av_kernel<false, V, X>), kc_grid(A.n), kAT, A, c, b, v, kc_parts(parts, A.n), st);
}
template <class X>
void amg_launch_kc_rt(hipStream_t s, int32_t n, const X *b, const X *v, const X *dinv, double *parts, X *rt, X *xa,
                      const PcgState *st) {
    ALAUNCH(kc_rt_kernel<X>, reduce_grid(n, kAT), kAT, n, b, v, dinv, kc_parts(parts, n), rt, xa, st);
}
template <class V, class X>
void amg_launch_kc_rt_resid(hipStream_t s, Sell<V> A, const X *b, const X *v, const X *dinv, double *parts, X *rt,
                            X *r, const PcgState *st) {
    ALAUNCH((kc_rt_resid_kernel<V, X>), grid_small(A.n), kAT, A, b, v, dinv, kc_parts(parts, A.n), rt, r, st);
}
template <class V, class X>
void amg_launch_kc_aw(hipStream_t s, Sell<V> A, const X *d, const X *v, const X *rt, double *parts,
                      const PcgState *st) {
    if (A.n <= kSmallRows)
        ALAUNCH((kc_aw_kernel<true, V, X>), kc_grid(A.n), kAT, A, d, v, rt, kc_parts(parts, A.n), st);
    else
        ALAUNCH((kc_aw_kernel<false, V, X>), kc_grid(A.n), kAT, A, d, v, rt, kc_parts(parts, A.n), st);
}
template <class X>
void amg_launch_kc_combine(hipStream_t s, int32_t n, const X *c, const X *d, double *parts, X *e,
                           const PcgState *st) {
    ALAUNCH(kc_combine_kernel<X>, reduce_grid(n, kAT), kAT, n, (KcE<X>{c, d, kc_parts(parts, n)}), e, st);
}
template <class V>
void amg_launch_update_resid(hipStream_t s, Sell<V> A, int k, double *x, const double *r_in, double *r_out,
                             const double *p, const double *q, const double *dinv, double *x0, double *res, PcgParts P,
                             PcgState *st) {
    ALAUNCH(pcg_update_resid_kernel<V>, krylov_shape(A.n).row_blocks, kSplitThreads, A, k, x, r_in, r_out, p, q, dinv, x0,
            res, P, st);
}
template <class V, class X>
void amg_launch_post_rz(hipStream_t s, Sell<V> A, const X *dinv, const X *b, const X *x, const int32_t *agg, const X *e,
                        const X *d, double *parts, int32_t nc, X *out, double *rz, double *zq, const X *qv,
                        const PcgState *st) {
    const KrylovShape ks = krylov_shape(A.n);
    ALAUNCH((vc_post_rz_kernel<V, X>), ks.row_blocks, kSplitThreads, A, ks.G, dinv, b, x, agg,
            (KcE<X>{e, d, kc_parts(parts, nc)}), out, rz, zq, qv, st);
}
#define KC_INST(V)                                                                                                    \
    template void amg_launch_kc_av<V, double>(hipStream_t, Sell<V>, const double *, const double *, double *, double *, \
                                              const PcgState *);                                                      \
    template void amg_launch_kc_rt_resid<V, double>(hipStream_t, Sell<V>, const double *, const double *,             \
                                                    const double *, double *, double *, double *, const PcgState *);  \
    template void amg_launch_kc_aw<V, double>(hipStream_t, Sell<V>, const double *, const double *, const double *,   \
                                              double *, const PcgState *);                                            \
    template void amg_launch_update_resid<V>(hipStream_t, Sell<V>, int, double *, const double *, double *,           \
                                             const double *, const double *, const double *, double *, double *,      \
                                             PcgParts, PcgState *);                                                   \
    template void amg_launch_post_rz<V, double>(hipStream_t, Sell<V>, const double *, const double *, const double *, \
                                                const int32_t *, const double *, const double *, double *, int32_t,   \
                                                double *, double *, double *, const double *, const PcgState *);
KC_INST(double)
KC_INST(float)
template void amg_launch_kc_rt<double>(hipStream_t, int32_t, const double *, const double *, const double *, double *,
                                       double *, double *, const PcgState *);
template void amg_launch_kc_combine<double>(hipStream_t, int32_t, const double *, const double *, double *, double *,
                                            const PcgState *);
template <class V, class X>
void amg_launch_pre(hipStream_t s, Sell<V> A, const X *dinv, const X *b, X *x, X *r, const PcgState *st) {
    ALAUNCH(vc_scale_kernel<X>, gridv(A.n), kAT, A.n, dinv, b, x, st);
    amg_launch_resid<V, X>(s, A, b, x, r, st);
}
template <class X>
void amg_launch_restrict(hipStream_t s, int32_t nc, const int32_t *mptr, const int32_t *mrows, const X *r, X *bc,
                         const X *dinv_c, X *xc, const PcgState *st) {
    ALAUNCH(vc_restrict_kernel<X>, gridv((int64_t)nc * kRL), kAT, nc, mptr, mrows, r, bc, dinv_c, xc, st);
}
template <class V, class X>
void amg_launch_resid(hipStream_t s, Sell<V> A, const X *b, const X *x, X *r, const PcgState *st) {
    if (A.n <= kSmallRows)
        ALAUNCH((vc_small_kernel<0, V, X>), grid_small(A.n), kAT, A, (const X *)nullptr, b, x, (const int32_t *)nullptr,
                (const X *)nullptr, r, st);
    else
        ALAUNCH((vc_resid_kernel<V, X>), gridv(A.n), kAT, A, b, x, r, st);
}
template <class V, class X>
void amg_launch_post_fused(hipStream_t s, Sell<V> A, const X *dinv, const X *b, const int32_t *agg, const X *e,
                           X *out, const PcgState *st) {
    if (A.n <= kSmallRows)
        ALAUNCH((vc_small_kernel<2, V, X>), grid_small(A.n), kAT, A, dinv, b, (const X *)nullptr, agg, e, out, st);
    else
        ALAUNCH((vc_post_fused_kernel<V, X>), gridv(A.n), kAT, A, dinv, b, agg, e, out, st);
}
template <class V, class X>
void amg_launch_post_x(hipStream_t s, Sell<V> A, const X *dinv, const X *b, const X *x, const int32_t *agg,
                       const X *e, X *out, const PcgState *st) {
    ALAUNCH((vc_small_kernel<3, V, X>), grid_small(A.n), kAT, A, dinv, b, x, agg, e, out, st);
}
template <class V, class X>
void amg_launch_post(hipStream_t s, Sell<V> A, const X *dinv, const X *b, const X *x, const int32_t *agg, const X *e,
                     X *y, X *out, double *rz, const PcgState *st, double *zq, const X *qv) {
    ALAUNCH(vc_prolong_kernel<X>, gridv(A.n), kAT, A.n, x, agg, e, y, st);
    // with rz the partials must match the Krylov kernels' grid and block size
    if (rz)
        ALAUNCH((vc_sweep_rz_kernel<V, X>), krylov_shape(A.n).row_blocks, kKrylovThreads, A, dinv, b, y, out, rz, zq, qv,
                st);
    else
        ALAUNCH((vc_sweep_kernel<V, X>), gridv(A.n), kAT, A, dinv, b, y, out, st);
}
template <class X>
void amg_launch_dense(hipStream_t s, int32_t n, const X *Ainv, const X *b, X *x, const PcgState *st) {
    ALAUNCH(vc_dense_kernel<X>, gridv((int64_t)n * 64), kAT, n, Ainv, b, x, st);
}
template <class V, class X>
void amg_launch_sweep(hipStream_t s, Sell<V> A, const X *dinv, const X *b, const X *x, X *out, const PcgState *st) {
    if (A.n <= kSmallRows)
        ALAUNCH((vc_small_kernel<1, V, X>), grid_small(A.n), kAT, A, dinv, b, x, (const int32_t *)nullptr,
                (const X *)nullptr, out, st);
    else
        ALAUNCH((vc_sweep_kernel<V, X>), gridv(A.n), kAT, A, dinv, b, x, out, st);
}
void launch_to_float(hipStream_t s, int64_t n, const double *a, float *b) {
    if (n > 0) ALAUNCH(to_float_kernel, gridv(n), kAT, n, a, b);
}
void launch_to_float_rowsum(hipStream_t s, Sell<double> A, float *v32, double *dg) {
    if (A.n > 0) ALAUNCH(to_float_rowsum_kernel, gridv(A.n), kAT, A, v32, dg);
}
void launch_to_double(hipStream_t s, int64_t n, const float *a, double *b) {
    if (n > 0) ALAUNCH(to_double_kernel, gridv(n), kAT, n, a, b);
}

#define VC_INST(V, X)                                                                                            \
    template void amg_launch_pre<V, X>(hipStream_t, Sell<V>, const X *, const X *, X *, X *, const PcgState *);    \
    template void amg_launch_resid<V, X>(hipStream_t, Sell<V>, const X *, const X *, X *, const PcgState *);       \
    template void amg_launch_post<V, X>(hipStream_t, Sell<V>, const X *, const X *, const X *, const int32_t *,    \
                                        const X *, X *, X *, double *, const PcgState *, double *, const X *);     \
    template void amg_launch_post_fused<V, X>(hipStream_t, Sell<V>, const X *, const X *, const int32_t *,         \
                                              const X *, X *, const PcgState *);                                   \
    template void amg_launch_post_x<V, X>(hipStream_t, Sell<V>, const X *, const X *, const X *, const int32_t *,  \
                                          const X *, X *, const PcgState *);                                       \
    template void amg_launch_sweep<V, X>(hipStream_t, Sell<V>, const X *, const X *, const X *, X *,               \
                                         const PcgState *);
VC_INST(double, double)
VC_INST(float, double)
VC_INST(float, float)
template void amg_launch_restrict<double>(hipStream_t, int32_t, const int32_t *, const int32_t *, const double *,
                                          double *, const double *, double *, const PcgState *);
template void amg_launch_restrict<float>(hipStream_t, int32_t, const int32_t *, const int32_t *, const float *,
                                         float *, const float *, float *, const PcgState *);
template void amg_launch_dense<double>(hipStream_t, int32_t, const double *, const double *, double *,
                                       const PcgState *);
template void amg_launch_dense<float>(hipStream_t, int32_t, const float *, const float *, float *, const PcgState *);
}  // namespace vag
