// Classical (Ruge-Stueben type) AMG hierarchy: the kernels (host side in
// amg_host.cpp).  The paper's solver study (§5.3) uses a classical AMG
// (BoomerAMG) beside aggregation AMG; this is the GPU form used here:
//
// * strength: j strongly influences i when -a_ij >= theta max_{k != i}(-a_ik)
//   (negative couplings only).  The matrices are symmetric, so whether i
//   strongly influences j is read from the same entry with j's row maximum,
//   and the measure lambda_i (how many points i influences) needs no
//   transpose;
// * coarse/fine splitting by PMIS (De Sterck, Yang, Heys): a point is coarse
//   when its key (lambda, then a bijective hash of the index) exceeds those
//   of all undecided strong neighbours; undecided points that strongly
//   depend on a new coarse point become fine; points that influence no one
//   start fine;
// * direct interpolation (Stueben's review of AMG): w_ij = -alpha_i a_ij / a~_ii
//   over the strong coarse neighbours, alpha_i = sum of all negative
//   couplings / sum of the strong coarse ones, a~_ii = a_ii + the positive
//   couplings;
// * R = P^T row by row (a coarse point's row lists the fine neighbours that
//   interpolate from it, in the order of its own matrix row: no atomics);
// * Galerkin product R (A P) by two sparse products, one wavefront per output
//   row accumulating in LDS in a fixed order (rows too wide for it: one
//   thread per row and an open-addressing table in a scratch buffer):
//   bitwise reproducible.
#include <algorithm>

#include "amg.h"
#include "reduce.h"
#include "sell.h"

namespace vag {

namespace {

constexpr int kCT = 256;
// undecided, coarse, fine; kN: coarse since this round's selection
constexpr int8_t kU = 0, kC = 1, kF = 2, kN = 3;

#define CL_GS(i, n) \
    for (int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); i < (n); i += (int32_t)(gridDim.x * blockDim.x))

int cgrid(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + kCT - 1) / kCT, 16384)); }

__device__ inline int sell_w(const int64_t *ptr, int32_t i) { return (int)((ptr[(i >> 6) + 1] - ptr[i >> 6]) >> 6); }
__device__ inline int64_t sell_at(const int64_t *ptr, int32_t i) { return ptr[i >> 6] + (i & 63); }

// bijective mixing of a 32-bit index (xorshift-multiply rounds, each invertible)
__device__ inline uint32_t mix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

}  // namespace

// (The kernels over matrix rows read eight slots ahead, row_slots: on the four
// levels of a 64^3 mesh the row maxima took 151 us and the strengths 135 one
// slot's chain of loads at a time, now 35 and 89.)
// m_i = max over off-diagonal entries of -a_ij (0 when none is negative)
__global__ __launch_bounds__(kCT) void cl_negmax_kernel(Sell<double> A, double *m) {
    CL_GS(i, A.n) {
        double mx = 0.0, v[kSlots];
        int32_t c[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t p) {
                c[j] = A.col[p];
                v[j] = A.val[p];
            },
            [&](int j, int64_t) {
                if (c[j] != i) mx = fmax(mx, -v[j]);
            });
        m[i] = mx;
    }
}

// per stored entry: bit 0 = i depends strongly on j, bit 1 = j depends
// strongly on i; keys and initial states; the rounds' counts cleared
__global__ __launch_bounds__(kCT) void cl_strength_kernel(Sell<double> A, const double *m, double theta, uint8_t *sf,
                                                          uint64_t *key, int8_t *state, int *counts) {
    CL_GS(k, kMisRounds) counts[k] = 0;
    CL_GS(i, A.n) {
        const double mi = m[i];
        uint32_t lam = 0;
        double v[kSlots], mj[kSlots];
        int32_t c[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t p) {
                c[j] = A.col[p];
                v[j] = -A.val[p];
                mj[j] = m[c[j]];
            },
            [&](int j, int64_t p) {
                uint8_t f = 0;
                if (c[j] != i && v[j] > 0.0) {
                    if (v[j] >= theta * mi) f |= 1;
                    if (v[j] >= theta * mj[j]) f |= 2;
                }
                sf[p] = f;
                lam += f >> 1;
            });
        key[i] = ((uint64_t)lam << 32) | mix32((uint32_t)i);
        state[i] = lam == 0 ? kF : kU;
    }
}

// Undecided points whose key beats every strong neighbour undecided at the
// round's start (kU or by now kN) become coarse.  progress (pinned): the round
// begun, or past kMisRounds when the last one (its count `last`, null in round
// 0) left nothing undecided; rounds from there on return at once.
__global__ __launch_bounds__(kCT) void cl_pmis_select_kernel(Sell<double> A, const uint8_t *sf, const uint64_t *key,
                                                             int8_t *st, int round, const int *last, int *progress) {
    const bool over = last && *last == 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) host_put(progress, over ? kMisRounds + 1 : round + 1);
    if (over) return;
    CL_GS(i, A.n) {
        if (st[i] != kU) continue;
        const uint64_t ki = key[i];
        bool top = true;
        int32_t c[kSlots];
        uint8_t f[kSlots];
        int8_t u[kSlots];
        uint64_t k[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t p) {
                c[j] = A.col[p];
                f[j] = sf[p];
                u[j] = st[c[j]];
                k[j] = key[c[j]];
            },
            [&](int j, int64_t) { top = top && !(f[j] && (u[j] == kU || u[j] == kN) && k[j] > ki); });
        if (top) st[i] = kN;
    }
}

// undecided points that depend strongly on a coarse point become fine; the
// remaining undecided points are counted (one atomic per block)
__global__ __launch_bounds__(kCT) void cl_pmis_fine_kernel(Sell<double> A, const uint8_t *sf, int8_t *st, int *cnt,
                                                           const int *last) {
    if (last && *last == 0) return;
    int mine = 0;
    CL_GS(i, A.n) {
        if (st[i] == kN) st[i] = kC;
        if (st[i] != kU) continue;
        bool fine = false, f[kSlots];
        row_slots(
            A.ptr, i,
            [&](int j, int64_t p) {
                const int8_t u = st[A.col[p]];
                f[j] = (sf[p] & 1) && (u == kC || u == kN);
            },
            [&](int j, int64_t) { fine = fine || f[j]; });
        if (fine)
            st[i] = kF;
        else
            ++mine;
    }
    const int total = __syncthreads_count(mine > 0) > 0 ? 1 : 0;
    if (threadIdx.x == 0 && total) atomicAdd(cnt, 1);
}

// points still undecided after the last round become coarse
__global__ __launch_bounds__(kCT) void cl_pmis_close_kernel(int32_t n, int8_t *st) {
    CL_GS(i, n) if (st[i] == kU) st[i] = kC;
}

// interpolation row lengths and coarse flags
__global__ __launch_bounds__(kCT) void cl_interp_count_kernel(Sell<double> A, const uint8_t *sf, const int8_t *st,
                                                              int32_t *plen, int32_t *cflag) {
    CL_GS(i, A.n) {
        if (st[i] == kC) {
            plen[i] = 1;
            cflag[i] = 1;
            continue;
        }
        cflag[i] = 0;
        int32_t c = 0;
        bool f[kSlots];
        row_slots(
            A.ptr, i, [&](int j, int64_t p) { f[j] = (sf[p] & 1) && st[A.col[p]] == kC; },
            [&](int j, int64_t) { c += f[j]; });
        plen[i] = c;
    }
}

__global__ __launch_bounds__(kCT) void cl_interp_fill_kernel(Sell<double> A, const uint8_t *sf, const int8_t *st,
                                                             const int32_t *cidx, const int32_t *pptr, int32_t *pcol,
                                                             double *pval, int32_t *cfine) {
    CL_GS(i, A.n) {
        int32_t q = pptr[i];
        if (st[i] == kC) {
            pcol[q] = cidx[i];
            pval[q] = 1.0;
            cfine[cidx[i]] = i;
            continue;
        }
        if (pptr[i + 1] == q) continue;
        double aii = 0.0, neg = 0.0, pos = 0.0, negc = 0.0, v[kSlots];
        int32_t c[kSlots];
        bool f[kSlots];
        auto load = [&](int j, int64_t p) {
            c[j] = A.col[p];
            v[j] = A.val[p];
            f[j] = (sf[p] & 1) && st[c[j]] == kC;
        };
        row_slots(A.ptr, i, load, [&](int j, int64_t) {
            if (c[j] == i) {
                aii += v[j];  // padding entries hold 0
            } else {
                neg += fmin(v[j], 0.0);
                pos += fmax(v[j], 0.0);
                if (f[j]) negc += v[j];
            }
        });
        const double scale = -(neg / negc) / (aii + pos);
        row_slots(A.ptr, i, load, [&](int j, int64_t) {
            if (c[j] != i && f[j]) {
                pcol[q] = cidx[c[j]];
                pval[q] = scale * v[j];
                ++q;
            }
        });
    }
}

// R = P^T: coarse point c (fine point f) takes (f, 1) and, for each fine
// neighbour i of f in A's row order, P's weight of c in row i
// (kTL lanes per coarse point, over the row's neighbours; one lane per point
// took 100 us at 57 k coarse points)
constexpr int kTL = 16;
template <bool FILL>
__global__ __launch_bounds__(kCT) void cl_transpose_kernel(Sell<double> A, int32_t nc, const int32_t *cfine,
                                                           const int8_t *st, const int32_t *pptr, const int32_t *pcol,
                                                           const double *pval, int32_t *rlen, const int32_t *rptr,
                                                           int32_t *rcol, double *rval) {
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int sub = threadIdx.x & (kTL - 1), shift = (threadIdx.x & 63) & ~(kTL - 1);
    const int32_t step = (int32_t)((int64_t)gridDim.x * blockDim.x / kTL);
    // every lane of a wavefront runs the same number of passes (the ballots need them all)
    for (int32_t cb = (int32_t)(t0 / kTL) - shift / kTL; cb < nc; cb += step) {
        const int32_t c = cb + shift / kTL;
        const int32_t f = c < nc ? cfine[c] : -1;
        int32_t q = FILL && f >= 0 ? rptr[c] : 0;
        if (FILL && f >= 0 && sub == 0) {
            rcol[q] = f;
            rval[q] = 1.0;
        }
        ++q;
        const int64_t b = f >= 0 ? sell_at(A.ptr, f) : 0;
        const int w = f >= 0 ? sell_w(A.ptr, f) : 0;
        for (int j0 = 0; __ballot(j0 < w); j0 += kTL) {
            int32_t i = -1, at = -1;
            if (j0 + sub < w) {
                i = A.col[b + (int64_t)(j0 + sub) * 64];
                if (i != f && st[i] != kC)
                    for (int32_t t = pptr[i]; t < pptr[i + 1]; ++t)
                        if (pcol[t] == c) {
                            at = t;
                            break;
                        }
            }
            const uint32_t mask = (uint32_t)(__ballot(at >= 0) >> shift) & ((1u << kTL) - 1);
            if (FILL && at >= 0) {
                const int32_t o = q + __popc(mask & ((1u << sub) - 1));
                rcol[o] = i;
                rval[o] = pval[at];
            }
            q += __popc(mask);
        }
        if (!FILL && f >= 0 && sub == 0) rlen[c] = q;
    }
}

// Table sizes of a product row: cap = the power of two >= 2 x (number of
// contributions), at least 8, at most kClCapMax (a row with more distinct
// columns than its table holds sets *overflow).
__device__ inline int32_t cl_cap(int64_t bound) {
    int64_t c = 8;
    while (c < 2 * bound && c < kClCapMax) c <<= 1;
    return (int32_t)c;
}

// contributions of row i of A P: sum over A's nonzero entries of |P row|
__global__ __launch_bounds__(kCT) void cl_ap_cap_kernel(Sell<double> A, const int32_t *pptr, const int32_t *big,
                                                        int32_t *cap) {
    CL_GS(i, A.n) {
        if (!big[i]) {
            cap[i] = 0;
            continue;
        }
        const int64_t b = sell_at(A.ptr, i);
        const int w = sell_w(A.ptr, i);
        int64_t s = 0;
        for (int j = 0; j < w; ++j) {
            const int64_t p = b + (int64_t)j * 64;
            if (A.val[p] != 0.0) s += pptr[A.col[p] + 1] - pptr[A.col[p]];
        }
        cap[i] = cl_cap(s);
    }
}

// contributions of row c of R (A P)
__global__ __launch_bounds__(kCT) void cl_rap_cap_kernel(int32_t nc, const int32_t *rptr, const int32_t *rcol,
                                                         const int32_t *apptr, const int32_t *big, int32_t *cap) {
    CL_GS(c, nc) {
        if (!big[c]) {
            cap[c] = 0;
            continue;
        }
        int64_t s = 0;
        for (int32_t q = rptr[c]; q < rptr[c + 1]; ++q) s += apptr[rcol[q] + 1] - apptr[rcol[q]];
        cap[c] = cl_cap(s);
    }
}

// sum of the table sizes of each chunk of kClChunk rows
__global__ __launch_bounds__(kCT) void cl_chunk_sum_kernel(int32_t n, const int32_t *cap, int64_t *sums) {
    const int32_t r0 = blockIdx.x * kClChunk, r1 = min(n, r0 + kClChunk);
    int64_t s = 0;
    for (int32_t i = r0 + threadIdx.x; i < r1; i += kCT) s += cap[i];
    __shared__ int64_t red[kCT];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = kCT / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = red[0];
}

// Products, one wavefront per output row (their rows are short: ~20 columns in
// A P, ~50 in R A P).  The distinct columns are found with an LDS hash set and
// put in the order of cl_product_kernel's table; the sums run in the order of X's entries, each over its row of Y, so
// the values do not depend on timing.  A row that outgrows the kernel's LDS is
// marked in big (and counted) and left to cl_product_kernel.  One thread per
// row with its table in global memory, as there, waits on a chain of dependent
// loads per contribution: 17 ms for the four levels of a 64^3 hierarchy,
// against 1.1 ms here, both passes of both products.
__device__ inline bool cl_insert(int32_t *keys, int mask, int32_t J, uint32_t &h) {
    h = mix32((uint32_t)J) & (uint32_t)mask;
    for (;;) {
        const int32_t prev = atomicCAS(&keys[h], -1, J);
        if (prev == -1) return true;
        if (prev == J) return false;
        h = (h + 1) & (uint32_t)mask;
    }
}

// The order of a row's columns is that of cl_product_kernel's table, which takes
// them by first contribution: cols[0 .. nd) in that order to a table of C slots
// (two 16-bit indices of cols per word of T, 0xffff an empty slot).  In linear
// probing the earlier column keeps a slot, so a column passes slots of earlier
// ones and sends later ones on from where they sit: any order of the lanes'
// steps ends in the same table.  C >= 2 nd, so every chain ends.
constexpr int kClTable = 4096;
__device__ inline void cl_place(uint32_t *T, int32_t C, const int32_t *cols, int nd, int lane) {
    for (int k = lane; k < C / 2; k += 64) T[k] = 0xffffffffu;
    __syncthreads();
    const int lg = 31 - __builtin_clz((unsigned)C);
    for (int k = lane; k < nd; k += 64) {
        uint32_t cur = (uint32_t)k, h = mix32((uint32_t)cols[k]) >> (32 - lg);
        for (;;) {
            const int sh = (int)(h & 1) * 16;
            uint32_t w = T[h >> 1], old;
            for (;;) {
                old = (w >> sh) & 0xffffu;
                if (old < cur) break;
                const uint32_t prev = atomicCAS(&T[h >> 1], w, (w & ~(0xffffu << sh)) | cur << sh);
                if (prev == w) break;
                w = prev;
            }
            if (old == 0xffffu) break;
            cur = max(cur, old);
            h = (h + 1) & (uint32_t)(C - 1);
        }
    }
    __syncthreads();
}
// f(position, index of cols) for the columns in the order of the slots
template <class F>
__device__ inline void cl_placed(const uint32_t *T, int32_t C, int lane, F f) {
    int n = 0;
    for (int k0 = 0; k0 < C; k0 += 64) {
        const int k = k0 + lane;
        const uint32_t v = k < C ? (T[k >> 1] >> (k & 1) * 16) & 0xffffu : 0xffffu;
        const uint64_t mask = __ballot(v != 0xffffu);
        if (v != 0xffffu) f(n + __popcll(mask & ((1ull << lane) - 1)), (int)v);
        n += __popcll(mask);
    }
}

// Row i of A P.  Up to kApCand contributions (A's entries times P's rows,
// flattened over the lanes; at most 195 on jittered hexahedra up to 40^3) are
// held in LDS; each lane then sums the columns
// it owns over all contributions in order.
constexpr int kApCand = 256, kApHash = 256, kApCols = 128;
template <bool FILL>
__global__ __launch_bounds__(64) void cl_ap_wave_kernel(int32_t r0, Sell<double> A, const int32_t *__restrict__ pptr,
                                                        const int32_t *__restrict__ pcol,
                                                        const double *__restrict__ pval, int32_t *__restrict__ big,
                                                        int *__restrict__ nbig, int32_t *__restrict__ rowlen,
                                                        const int64_t *__restrict__ optr, int32_t *__restrict__ ocol,
                                                        double *__restrict__ oval) {
    __shared__ int32_t cj[kApCand], keys[kApHash], cols[kApCols], sorted[kApCols];
    __shared__ double cv[FILL ? kApCand : 1], xs[64];
    __shared__ int first[FILL ? kApHash : 1];  // contribution to each key
    __shared__ uint8_t hs[FILL ? kApCand : 1];
    __shared__ uint32_t T[FILL ? kApCand : 1];
    __shared__ int32_t off[65], y0[64];
    const int32_t i = r0 + (int32_t)blockIdx.x;
    const int lane = threadIdx.x;
    if (FILL && big[i]) return;
    for (int k = lane; k < kApHash; k += 64) {
        keys[k] = -1;
        if (FILL) first[k] = kApCand;
    }
    const int64_t b = sell_at(A.ptr, i);
    const int w = sell_w(A.ptr, i);
    int m = 0, nd = 0;
    bool over = false;
    for (int j0 = 0; j0 < w && !over; j0 += 64) {
        const int j = j0 + lane;
        double x = 0.0;
        int32_t t = 0;
        if (j < w) {
            x = A.val[b + (int64_t)j * 64];
            t = A.col[b + (int64_t)j * 64];
        }
        const int32_t p = pptr[t];
        const int c = x != 0.0 ? pptr[t + 1] - p : 0;
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        const int tot = __shfl(incl, 63, 64);
        over = m + tot > kApCand;
        if (over) break;
        __syncthreads();
        off[lane] = incl - c;
        if (lane == 0) off[64] = tot;
        y0[lane] = p;
        xs[lane] = x;
        __syncthreads();
        for (int e0 = 0; e0 < tot; e0 += 64) {
            const int e = e0 + lane;
            bool fresh = false;
            if (e < tot) {
                int lo = 0, hi = 63;  // the last entry whose first contribution is at or before e
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (off[mid] <= e) lo = mid; else hi = mid - 1;
                }
                const int32_t q = y0[lo] + e - off[lo], J = pcol[q];
                cj[m + e] = J;
                if (FILL) cv[m + e] = xs[lo] * pval[q];
                uint32_t h;
                fresh = cl_insert(keys, kApHash - 1, J, h);
                if (FILL) {
                    hs[m + e] = (uint8_t)h;
                    atomicMin(&first[h], m + e);
                }
            }
            nd += __popcll(__ballot(fresh));
            over = over || nd > kApCols;
            if (over) break;
        }
        m += tot;
    }
    if (!FILL) {
        if (lane == 0) {
            rowlen[i] = over ? 0 : nd;
            big[i] = over;
            if (over) atomicAdd(nbig, 1);
        }
        return;
    }
    __syncthreads();
    int nc = 0;
    for (int e0 = 0; e0 < m; e0 += 64) {
        const int e = e0 + lane;
        const bool is = e < m && first[hs[e]] == e;
        const uint64_t mask = __ballot(is);
        if (is) cols[nc + __popcll(mask & ((1ull << lane) - 1))] = cj[e];
        nc += __popcll(mask);
    }
    __syncthreads();
    const int32_t C = cl_cap(m);  // at most 2 kApCand
    cl_place(T, C, cols, nd, lane);
    cl_placed(T, C, lane, [&](int k, int v) { sorted[k] = cols[v]; });
    __syncthreads();
    const int64_t o = optr[i];
    for (int k = lane; k < nd; k += 64) {
        const int32_t J = sorted[k];
        double s = 0.0;
#pragma unroll 8
        for (int e = 0; e < m; ++e) s += cj[e] == J ? cv[e] : 0.0;
        ocol[o + k] = J;
        oval[o + k] = s;
    }
}

// Row c of R (A P): R's entries one after the other, the lanes over the
// columns of that entry's row of A P (distinct columns, so no two lanes add to
// the same sum), the next row's columns loaded meanwhile.  Up to kRapCols
// distinct columns (at most 93 on those meshes).
constexpr int kRapHash = 512, kRapCols = 256;
template <bool FILL>
__global__ __launch_bounds__(64) void cl_rap_wave_kernel(int32_t r0, const int32_t *__restrict__ xptr,
                                                         const int32_t *__restrict__ xcol,
                                                         const double *__restrict__ xval,
                                                         const int32_t *__restrict__ yptr,
                                                         const int32_t *__restrict__ ycol,
                                                         const double *__restrict__ yval, int32_t *__restrict__ big,
                                                         int *__restrict__ nbig, int32_t *__restrict__ rowlen,
                                                         const int64_t *__restrict__ optr, int32_t *__restrict__ ocol,
                                                         double *__restrict__ oval) {
    __shared__ uint32_t T[FILL ? kClTable / 2 : kRapHash];  // of cl_place; before that the keys
    int32_t *keys = reinterpret_cast<int32_t *>(T);
    __shared__ int32_t cols[FILL ? kRapCols : 1];
    __shared__ double sums[FILL ? kRapHash : 1], xs[64];
    __shared__ uint16_t slot[FILL ? kRapCols : 1];
    __shared__ int32_t lo[64], hi[64];
    const int32_t c = r0 + (int32_t)blockIdx.x;
    const int lane = threadIdx.x;
    if (FILL && big[c]) return;
    for (int k = lane; k < kRapHash; k += 64) {
        keys[k] = -1;
        if (FILL) sums[k] = 0.0;
    }
    int nd = 0, m = 0;
    bool over = false;
    const int32_t a1 = xptr[c + 1];
    for (int32_t a0 = xptr[c]; a0 < a1 && !over; a0 += 64) {
        __syncthreads();
        if (a0 + lane < a1) {
            const int32_t t = xcol[a0 + lane];
            lo[lane] = yptr[t];
            hi[lane] = yptr[t + 1];
            if (FILL) xs[lane] = xval[a0 + lane];
            m += hi[lane] - lo[lane];
        }
        __syncthreads();
        const int na = min(64, (int)(a1 - a0));
        int32_t J = lo[0] + lane < hi[0] ? ycol[lo[0] + lane] : -1;
        double v = FILL && J >= 0 ? yval[lo[0] + lane] : 0.0;
        for (int k = 0; k < na && !over; ++k) {
            const int32_t e = hi[k];
            const double x = FILL ? xs[k] : 0.0;
            int32_t Jn = -1;  // the first columns of the next row
            double vn = 0.0;
            if (k + 1 < na && lo[k + 1] + lane < hi[k + 1]) {
                Jn = ycol[lo[k + 1] + lane];
                if (FILL) vn = yval[lo[k + 1] + lane];
            }
            for (int32_t q = lo[k] + lane;;) {
                bool fresh = false;
                uint32_t h = 0;
                if (J >= 0) {
                    fresh = cl_insert(keys, kRapHash - 1, J, h);
                    if (FILL) {
#pragma clang fp contract(off)  // as cl_product_kernel's sums
                        const double t = x * v;
                        sums[h] = sums[h] + t;
                    }
                }
                const uint64_t mask = __ballot(fresh);
                if (FILL && fresh) {  // by first contribution; nd <= kRapCols as counted
                    const int at = nd + __popcll(mask & ((1ull << lane) - 1));
                    cols[at] = J;
                    slot[at] = (uint16_t)h;
                }
                nd += __popcll(mask);
                over = over || nd > kRapCols;
                q += 64;
                if (over || __ballot(q < e) == 0) break;
                J = q < e ? ycol[q] : -1;
                v = FILL && J >= 0 ? yval[q] : 0.0;
            }
            __syncthreads();
            J = Jn;
            v = vn;
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m += __shfl_xor(m, d, 64);
    const int32_t C = cl_cap(m);
    over = over || C > kClTable;
    if (!FILL) {
        if (lane == 0) {
            rowlen[c] = over ? 0 : nd;
            big[c] = over;
            if (over) atomicAdd(nbig, 1);
        }
        return;
    }
    __syncthreads();
    cl_place(T, C, cols, nd, lane);
    const int64_t o = optr[c >> 6] + (c & 63);
    cl_placed(T, C, lane, [&](int k, int v) {
        ocol[o + (int64_t)k * 64] = cols[v];
        oval[o + (int64_t)k * 64] = sums[slot[v]];
    });
    const int w = sell_w(optr, c);  // padding of the slice: the row itself with value 0
    for (int k = nd + lane; k < w; k += 64) {
        ocol[o + (int64_t)k * 64] = c;
        oval[o + (int64_t)k * 64] = 0.0;
    }
}

// The rows the wavefront kernels leave (big), one per thread: accumulate
// sum_t x_it * (row t of Y) into the
// row's own table (slots hoff[i - r0] .. + cap[i]), then either count the
// distinct columns (rowlen) or write them in slot order.  X is A in sliced
// ELL (SELL_X) or R in CSR; the output is CSR (optr) or sliced ELL (SELL_OUT).
template <bool SELL_X, bool SELL_OUT>
__global__ __launch_bounds__(kCT) void cl_product_kernel(int32_t r0, int32_t r1, Sell<double> AX, const int32_t *xptr,
                                                         const int32_t *xcol, const double *xval, const int32_t *yptr,
                                                         const int32_t *ycol, const double *yval, const int32_t *cap,
                                                         const int32_t *hoff, int32_t *hkey, double *hval,
                                                         const int32_t *big, int fill, int32_t *rowlen, const int64_t *optr,
                                                         int32_t *ocol, double *oval, int *overflow) {
    for (int32_t i = r0 + (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); i < r1;
         i += (int32_t)(gridDim.x * blockDim.x)) {
        if (!big[i]) continue;
        const int32_t C = cap[i];
        int32_t *K = hkey + hoff[i - r0];
        double *V = hval + hoff[i - r0];
        for (int32_t s = 0; s < C; ++s) K[s] = -1;
        const int lg = 31 - __builtin_clz((unsigned)C);
        bool over = false;
        auto add = [&](int32_t m, double v) {
            uint32_t h = (mix32((uint32_t)m) >> (32 - lg));
            for (int32_t probe = 0; probe < C; ++probe) {
                const int32_t k = K[h];
                if (k == m) {
                    V[h] += v;
                    return;
                }
                if (k == -1) {
                    K[h] = m;
                    V[h] = v;
                    return;
                }
                h = (h + 1) & (uint32_t)(C - 1);
            }
            over = true;
        };
        if (SELL_X) {
            const int64_t b = sell_at(AX.ptr, i);
            const int w = sell_w(AX.ptr, i);
            for (int j = 0; j < w && !over; ++j) {
                const int64_t p = b + (int64_t)j * 64;
                const double x = AX.val[p];
                if (x == 0.0) continue;
                const int32_t t = AX.col[p];
                for (int32_t q = yptr[t]; q < yptr[t + 1]; ++q) add(ycol[q], x * yval[q]);
            }
        } else {
            for (int32_t a = xptr[i]; a < xptr[i + 1] && !over; ++a) {
                const double x = xval[a];
                const int32_t t = xcol[a];
                for (int32_t q = yptr[t]; q < yptr[t + 1]; ++q) add(ycol[q], x * yval[q]);
            }
        }
        if (over) {
            *overflow = 1;
            if (!fill) rowlen[i] = 0;
            continue;
        }
        if (!fill) {
            int32_t n = 0;
            for (int32_t s = 0; s < C; ++s) n += K[s] != -1;
            rowlen[i] = n;
        } else {
            int32_t j = 0;
            for (int32_t s = 0; s < C; ++s) {
                if (K[s] == -1) continue;
                const int64_t p = SELL_OUT ? optr[i >> 6] + (int64_t)j * 64 + (i & 63) : optr[i] + j;
                ocol[p] = K[s];
                oval[p] = V[s];
                ++j;
            }
            if (SELL_OUT) {  // padding of the slice: the row itself with value 0
                const int w = (int)((optr[(i >> 6) + 1] - optr[i >> 6]) >> 6);
                for (; j < w; ++j) {
                    const int64_t p = optr[i >> 6] + (int64_t)j * 64 + (i & 63);
                    ocol[p] = i;
                    oval[p] = 0.0;
                }
            }
        }
    }
}

// cycle: bc = R r (and xc = D_c^-1 bc); y = x + P e.  R's rows hold 5 to 20
// entries: kRLanes lanes load and gather, and the row's sum runs over them in the
// order of the entries (one lane per row waited on its chain of gathers: 10 us
// per visit at 57 k rows)
constexpr int kRLanes = 8;
template <class X>
__global__ __launch_bounds__(kCT) void cl_restrict_kernel(int32_t nc, const int32_t *rptr, const int32_t *rcol,
                                                          const double *rval, const X *r, X *bc, const X *dinv_c,
                                                          X *xc, const PcgState *st) {
    if (st && st->done) return;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int sub = threadIdx.x & (kRLanes - 1), g = (threadIdx.x & 63) / kRLanes;
    const int64_t step = (int64_t)gridDim.x * blockDim.x / kRLanes;
    // every lane of a wavefront runs the same number of passes (the shuffles need them all)
    for (int64_t cb = t0 / kRLanes - g; cb < nc; cb += step) {
        const int64_t c = cb + g;
        const int32_t q1 = c < nc ? rptr[c + 1] : 0;
        double s = 0.0;
        for (int32_t q = c < nc ? rptr[c] : 0; __ballot(q < q1); q += kRLanes) {
            const bool on = q + sub < q1;
            const double v = on ? rval[q + sub] : 0.0, x = on ? (double)r[rcol[q + sub]] : 0.0;
#pragma unroll
            for (int k = 0; k < kRLanes; ++k) {
                const double t = fma(__shfl(v, k, kRLanes), __shfl(x, k, kRLanes), s);
                s = q + k < q1 ? t : s;
            }
        }
        if (sub == 0 && c < nc) {
            bc[c] = (X)s;
            if (xc) xc[c] = dinv_c[c] * (X)s;
        }
    }
}

template <class X>
__global__ __launch_bounds__(kCT) void cl_prolong_kernel(int32_t n, const int32_t *pptr, const int32_t *pcol,
                                                         const double *pval, const X *x, const X *e, X *y,
                                                         const PcgState *st) {
    if (st && st->done) return;
    CL_GS(i, n) {
        double s = (double)x[i];
        for (int32_t q = pptr[i]; q < pptr[i + 1]; ++q) s += pval[q] * (double)e[pcol[q]];
        y[i] = (X)s;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define CLAUNCH(kern, grid, ...)                                                  \
    do {                                                                          \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kCT), 0, s, __VA_ARGS__);       \
        VAG_HIP(hipGetLastError());                                               \
    } while (0)

void cl_launch_strength(hipStream_t s, Sell<double> A, double theta, double *m, uint8_t *sf, uint64_t *key,
                        int8_t *state, int *counts) {
    if (A.n <= 0) return;
    CLAUNCH(cl_negmax_kernel, cgrid(A.n), A, m);
    CLAUNCH(cl_strength_kernel, cgrid(A.n), A, m, theta, sf, key, state, counts);
}
void cl_launch_pmis(hipStream_t s, Sell<double> A, const uint8_t *sf, const uint64_t *key, int8_t *st, int *counts,
                    int *progress) {
    if (A.n <= 0) return;
    volatile int *started = progress;
    *started = 0;
    for (int r = 0; r < kMisRounds; ++r) {
        const int *last = r ? counts + r - 1 : nullptr;
        CLAUNCH(cl_pmis_select_kernel, cgrid(A.n), A, sf, key, st, r, last, progress);
        CLAUNCH(cl_pmis_fine_kernel, cgrid(A.n), A, sf, st, counts + r, last);
        poll_rounds(s, started, r - 2, kMisRounds);
        if (*started > kMisRounds) return;
    }
    CLAUNCH(cl_pmis_close_kernel, cgrid(A.n), A.n, st);
}
void cl_launch_interp_count(hipStream_t s, Sell<double> A, const uint8_t *sf, const int8_t *st, int32_t *plen,
                            int32_t *cflag) {
    if (A.n > 0) CLAUNCH(cl_interp_count_kernel, cgrid(A.n), A, sf, st, plen, cflag);
}
void cl_launch_interp_fill(hipStream_t s, Sell<double> A, const uint8_t *sf, const int8_t *st, const int32_t *cidx,
                           const int32_t *pptr, int32_t *pcol, double *pval, int32_t *cfine) {
    if (A.n > 0) CLAUNCH(cl_interp_fill_kernel, cgrid(A.n), A, sf, st, cidx, pptr, pcol, pval, cfine);
}
void cl_launch_transpose(hipStream_t s, Sell<double> A, int32_t nc, const int32_t *cfine, const int8_t *st,
                         const int32_t *pptr, const int32_t *pcol, const double *pval, int32_t *rlen,
                         const int32_t *rptr, int32_t *rcol, double *rval) {
    if (nc <= 0) return;
    if (!rptr)
        CLAUNCH(cl_transpose_kernel<false>, cgrid((int64_t)nc * kTL), A, nc, cfine, st, pptr, pcol, pval, rlen, rptr, rcol, rval);
    else
        CLAUNCH(cl_transpose_kernel<true>, cgrid((int64_t)nc * kTL), A, nc, cfine, st, pptr, pcol, pval, rlen, rptr, rcol, rval);
}
void cl_launch_ap_cap(hipStream_t s, Sell<double> A, const int32_t *pptr, const int32_t *big, int32_t *cap) {
    if (A.n > 0) CLAUNCH(cl_ap_cap_kernel, cgrid(A.n), A, pptr, big, cap);
}
void cl_launch_rap_cap(hipStream_t s, int32_t nc, const int32_t *rptr, const int32_t *rcol, const int32_t *apptr,
                       const int32_t *big, int32_t *cap) {
    if (nc > 0) CLAUNCH(cl_rap_cap_kernel, cgrid(nc), nc, rptr, rcol, apptr, big, cap);
}
void cl_launch_chunk_sums(hipStream_t s, int32_t n, const int32_t *cap, int64_t *sums) {
    if (n > 0) CLAUNCH(cl_chunk_sum_kernel, (n + kClChunk - 1) / kClChunk, n, cap, sums);
}
void cl_launch_product(hipStream_t s, int32_t r0, int32_t r1, const Sell<double> *AX, const int32_t *xptr,
                       const int32_t *xcol, const double *xval, const int32_t *yptr, const int32_t *ycol,
                       const double *yval, const int32_t *cap, const int32_t *hoff, int32_t *hkey, double *hval,
                       const int32_t *big, bool fill, int32_t *rowlen, const int64_t *optr, bool sell_out, int32_t *ocol, double *oval,
                       int *overflow) {
    if (r1 <= r0) return;
    const int g = cgrid(r1 - r0);
    const Sell<double> ax = AX ? *AX : Sell<double>{};
    if (AX && !sell_out)
        CLAUNCH((cl_product_kernel<true, false>), g, r0, r1, ax, xptr, xcol, xval, yptr, ycol, yval, cap, hoff, hkey,
                hval, big, fill ? 1 : 0, rowlen, optr, ocol, oval, overflow);
    else if (!AX && sell_out)
        CLAUNCH((cl_product_kernel<false, true>), g, r0, r1, ax, xptr, xcol, xval, yptr, ycol, yval, cap, hoff, hkey,
                hval, big, fill ? 1 : 0, rowlen, optr, ocol, oval, overflow);
    else
        throw Error(VAG_ERR_ARG, "internal: unsupported sparse product layout");
}
void cl_launch_product_rows(hipStream_t s, int32_t n, const Sell<double> *AX, const int32_t *xptr,
                            const int32_t *xcol, const double *xval, const int32_t *yptr, const int32_t *ycol,
                            const double *yval, int32_t *big, int *nbig, bool fill, int32_t *rowlen,
                            const int64_t *optr, int32_t *ocol, double *oval) {
    if (n <= 0) return;
    // a launch has fewer than 2^32 threads
    constexpr int32_t kRows = 1 << 25;
#define CL_ROWS(kern, ...)                                                                                   \
    do {                                                                                                     \
        for (int32_t r0 = 0; r0 < n; r0 += std::min(kRows, n - r0)) {                                        \
            const dim3 grid((unsigned)std::min(kRows, n - r0));                                              \
            if (fill)                                                                                        \
                hipLaunchKernelGGL((kern<true>), grid, dim3(64), 0, s, r0, __VA_ARGS__, yptr, ycol, yval, big, \
                                   nbig, rowlen, optr, ocol, oval);                                          \
            else                                                                                             \
                hipLaunchKernelGGL((kern<false>), grid, dim3(64), 0, s, r0, __VA_ARGS__, yptr, ycol, yval, big, \
                                   nbig, rowlen, optr, ocol, oval);                                          \
            VAG_HIP(hipGetLastError());                                                                      \
        }                                                                                                    \
    } while (0)
    if (AX)
        CL_ROWS(cl_ap_wave_kernel, *AX);
    else
        CL_ROWS(cl_rap_wave_kernel, xptr, xcol, xval);
#undef CL_ROWS
}
template <class X>
void cl_launch_restrict(hipStream_t s, int32_t nc, const int32_t *rptr, const int32_t *rcol, const double *rval,
                        const X *r, X *bc, const X *dinv_c, X *xc, const PcgState *st) {
    if (nc > 0) CLAUNCH(cl_restrict_kernel<X>, cgrid((int64_t)nc * kRLanes), nc, rptr, rcol, rval, r, bc, dinv_c, xc, st);
}
template <class X>
void cl_launch_prolong(hipStream_t s, int32_t n, const int32_t *pptr, const int32_t *pcol, const double *pval,
                       const X *x, const X *e, X *y, const PcgState *st) {
    if (n > 0) CLAUNCH(cl_prolong_kernel<X>, cgrid(n), n, pptr, pcol, pval, x, e, y, st);
}
template void cl_launch_restrict<double>(hipStream_t, int32_t, const int32_t *, const int32_t *, const double *,
                                         const double *, double *, const double *, double *, const PcgState *);
template void cl_launch_restrict<float>(hipStream_t, int32_t, const int32_t *, const int32_t *, const double *,
                                        const float *, float *, const float *, float *, const PcgState *);
template void cl_launch_prolong<double>(hipStream_t, int32_t, const int32_t *, const int32_t *, const double *,
                                        const double *, const double *, double *, const PcgState *);
template void cl_launch_prolong<float>(hipStream_t, int32_t, const int32_t *, const int32_t *, const double *,
                                       const float *, const float *, float *, const PcgState *);

}  // namespace vag
