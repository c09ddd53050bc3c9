// Block-Jacobi ILU(0): host symbolic phase, factorization and triangular
// solves (§5.3's block Jacobi ILU(0) preconditioner; blocks and elimination
// order are stated in ilu.h).
//
// One wavefront per block.  Inside a block the rows are visited by levels of
// the dependency graph (a row's level is one more than the highest level of
// the rows it depends on), so the rows of one level are independent: the
// factorization and the forward solve follow the lower-triangle graph, the
// backward solve the upper one.  The solve keeps the block's vector in LDS.
#include <algorithm>
#include <atomic>
#include <exception>
#include <thread>

#include "host_parallel.h"
#include "ilu.h"

namespace vag {

namespace {

constexpr int kIluThreads = 64;

template <class T>
void put(hipStream_t s, Tracker &tr, DBuf<T> &d, const std::vector<T> &v) {
    d.alloc(std::max<size_t>(v.size(), 1), tr);
    if (!v.empty()) VAG_HIP(hipMemcpyAsync(d.p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s));
}

// Levels of one block (natural rows [r0, r1)): forward uses the entries left
// of the diagonal, backward those right of it.  Fills the block's slice of
// rows (r0-based) and its level pointers (absolute offsets into rows).
void block_levels(const std::vector<int32_t> &fptr, const std::vector<uint16_t> &fcol,
                  const std::vector<int32_t> &fdiag, int32_t r0, int32_t r1, bool forward, std::vector<int32_t> &lev,
                  std::vector<int32_t> &rows, std::vector<int32_t> &lptr) {
    const int32_t m = r1 - r0;
    int32_t top = 0;
    if (forward) {
        for (int32_t i = 0; i < m; ++i) {
            const int32_t o = r0 + i;
            int32_t l = 0;
            for (int32_t p = fptr[o]; p < fdiag[o]; ++p) l = std::max(l, lev[r0 + fcol[p]] + 1);
            lev[o] = l;
            top = std::max(top, l);
        }
    } else {
        for (int32_t i = m - 1; i >= 0; --i) {
            const int32_t o = r0 + i;
            int32_t l = 0;
            for (int32_t p = fdiag[o] + 1; p < fptr[o + 1]; ++p) l = std::max(l, lev[r0 + fcol[p]] + 1);
            lev[o] = l;
            top = std::max(top, l);
        }
    }
    // counting sort of the block's rows by level (ascending row inside a level)
    std::vector<int32_t> cnt(top + 2, 0);
    for (int32_t i = 0; i < m; ++i) ++cnt[lev[r0 + i] + 1];
    for (int32_t l = 0; l <= top; ++l) cnt[l + 1] += cnt[l];
    for (int32_t l = 0; l <= top; ++l) lptr.push_back(r0 + cnt[l]);
    for (int32_t i = 0; i < m; ++i) rows[r0 + cnt[lev[r0 + i]]++] = r0 + i;
}

}  // namespace

__global__ void ilu_solve_lds_kernel(IluArgs g, IluLds L, const double *__restrict__ r, double *__restrict__ z,
                                     const PcgState *st);

void Ilu::build(hipStream_t s, Tracker &tr, const Symbolic &S, int B) {
    const int32_t n = S.nunk;
    if (B < 1 || B > kIluMaxBlock) throw Error(VAG_ERR_ARG, "ilu_block_rows out of range");
    const int32_t nblk = (n + B - 1) / B;
    // in-block entries of each natural row, by local column
    std::vector<int32_t> cnt(n), fptr((size_t)n + 1, 0);
    parallel_chunks(n, [&](int, int64_t o0, int64_t o1) {
        for (int64_t o = o0; o < o1; ++o) {
            const int32_t r = S.sys_new[o], b0 = (int32_t)(o / B) * B;
            int32_t c = 0;
            for (int32_t q = S.row_ptr[r]; q < S.row_ptr[r + 1]; ++q) {
                const int32_t co = S.sys_old[S.col[q]];
                c += co >= b0 && co < b0 + B;
            }
            cnt[o] = c;
        }
    }, 4096);
    for (int32_t o = 0; o < n; ++o) fptr[o + 1] = fptr[o] + cnt[o];
    const int64_t nent = fptr[n];
    std::vector<uint16_t> fcol(nent);
    std::vector<int32_t> fsrc(nent), fdiag(n), rdev(n);
    std::atomic<bool> nodiag{false};
    parallel_chunks(n, [&](int, int64_t o0, int64_t o1) {
        std::vector<std::pair<int32_t, int32_t>> e;
        for (int64_t o = o0; o < o1; ++o) {
            const int32_t r = S.sys_new[o], b0 = (int32_t)(o / B) * B;
            const int64_t base = S.sell_ptr[r / kSliceRows] + r % kSliceRows;
            e.clear();
            for (int32_t q = S.row_ptr[r]; q < S.row_ptr[r + 1]; ++q) {
                const int32_t co = S.sys_old[S.col[q]];
                if (co >= b0 && co < b0 + B)
                    e.emplace_back(co - b0, (int32_t)(base + (int64_t)(q - S.row_ptr[r]) * kSliceRows));
            }
            std::sort(e.begin(), e.end());
            int32_t d = -1;
            for (size_t k = 0; k < e.size(); ++k) {
                fcol[fptr[o] + k] = (uint16_t)e[k].first;
                fsrc[fptr[o] + k] = e[k].second;
                if (e[k].first == o - b0) d = fptr[o] + (int32_t)k;
            }
            if (d < 0) nodiag.store(true);
            fdiag[o] = d;
            rdev[o] = r;
        }
    }, 4096);
    if (nodiag.load()) throw Error(VAG_ERR_ARG, "internal: a system row has no diagonal entry");
    // level schedules, block by block
    std::vector<int32_t> lev(n), rows_f(n), rows_b(n);
    std::vector<std::vector<int32_t>> lf(nblk), lb(nblk);
    parallel_chunks(nblk, [&](int, int64_t b0, int64_t b1) {
        for (int64_t b = b0; b < b1; ++b) {
            const int32_t r0 = (int32_t)b * B, r1 = std::min<int32_t>(n, r0 + B);
            block_levels(fptr, fcol, fdiag, r0, r1, true, lev, rows_f, lf[b]);
            block_levels(fptr, fcol, fdiag, r0, r1, false, lev, rows_b, lb[b]);
        }
    }, 8);
    std::vector<int32_t> lvb_f(nblk + 1, 0), lvb_b(nblk + 1, 0), lptr_f, lptr_b;
    for (int32_t b = 0; b < nblk; ++b) {
        lvb_f[b + 1] = lvb_f[b] + (int32_t)lf[b].size();
        lvb_b[b + 1] = lvb_b[b] + (int32_t)lb[b].size();
        lptr_f.insert(lptr_f.end(), lf[b].begin(), lf[b].end());
        lptr_b.insert(lptr_b.end(), lb[b].begin(), lb[b].end());
    }
    lptr_f.push_back(n);
    lptr_b.push_back(n);
    std::vector<int4> slot_f(n), slot_b(n);
    for (int32_t t = 0; t < n; ++t) {
        const int32_t of = rows_f[t], ob = rows_b[t];
        slot_f[t] = make_int4(of - (of / B) * B, fptr[of], fdiag[of], 0);
        slot_b[t] = make_int4(ob - (ob / B) * B, fdiag[ob], fptr[ob + 1], 0);
    }
    nlev_ = std::max(lvb_f[nblk], lvb_b[nblk]);
    lds_ = IluLds{};
    lds_.rows = std::min(B, n);
    for (int32_t b = 0; b < nblk; ++b) {
        const int32_t r0 = b * B, r1 = std::min(n, r0 + B);
        lds_.ents = std::max(lds_.ents, fptr[r1] - fptr[r0]);
        lds_.levs = std::max(lds_.levs, std::max(lvb_f[b + 1] - lvb_f[b], lvb_b[b + 1] - lvb_b[b]));
    }
    put(s, tr, fptr_, fptr);
    put(s, tr, fcol_, fcol);
    put(s, tr, fsrc_, fsrc);
    put(s, tr, fdiag_, fdiag);
    put(s, tr, rdev_, rdev);
    put(s, tr, lvb_f_, lvb_f);
    put(s, tr, lptr_f_, lptr_f);
    put(s, tr, rows_f_, rows_f);
    put(s, tr, lvb_b_, lvb_b);
    put(s, tr, lptr_b_, lptr_b);
    put(s, tr, rows_b_, rows_b);
    put(s, tr, slot_f_, slot_f);
    put(s, tr, slot_b_, slot_b);
    fval_.alloc(std::max<int64_t>(nent, 1), tr);
    in_lds_ = lds_.pays(nblk);
    if (in_lds_)  // the kernel's limit is the process's, so the most that any handle asks for
        VAG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(ilu_solve_lds_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)IluLds::kMax));
    VAG_HIP(hipStreamSynchronize(s));  // the host vectors go out of scope
    nent_ = nent;
    B_ = B;
    a_ = IluArgs{n,          B,         nblk,      fptr_.p,   fcol_.p,   fsrc_.p,   fdiag_.p,  rdev_.p,
                 lvb_f_.p,   lptr_f_.p, rows_f_.p, lvb_b_.p,  lptr_b_.p, rows_b_.p, slot_f_.p, slot_b_.p,
                 fval_.p};
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kIluThreads) void ilu_factor_kernel(IluArgs g, const double *__restrict__ A,
                                                                 int *bad) {
    const int32_t b = blockIdx.x, r0 = b * g.B, r1 = min(g.n, r0 + g.B);
    const int tid = threadIdx.x;
    for (int32_t e = g.fptr[r0] + tid; e < g.fptr[r1]; e += kIluThreads) g.fval[e] = A[g.fsrc[e]];
    __syncthreads();
    for (int32_t l = g.lvb_f[b]; l < g.lvb_f[b + 1]; ++l) {
        for (int32_t t = g.lptr_f[l] + tid; t < g.lptr_f[l + 1]; t += kIluThreads) {
            const int32_t o = g.rows_f[t], p1 = g.fptr[o + 1], pd = g.fdiag[o];
            // subtract multiples of the final rows k < o, in increasing k,
            // at the positions row o stores
            for (int32_t p = g.fptr[o]; p < pd; ++p) {
                const int32_t k = r0 + g.fcol[p], dk = g.fdiag[k], k1 = g.fptr[k + 1];
                const double lik = g.fval[p] / g.fval[dk];
                g.fval[p] = lik;
                int32_t pp = p + 1;
                for (int32_t q = dk + 1; q < k1 && pp < p1; ++q) {
                    const uint16_t j = g.fcol[q];
                    while (pp < p1 && g.fcol[pp] < j) ++pp;
                    if (pp < p1 && g.fcol[pp] == j) g.fval[pp] -= lik * g.fval[q];
                }
            }
            const double d = g.fval[pd];
            if (!(d != 0.0) || !__builtin_isfinite(d)) *bad = 1 + o;
        }
        __syncthreads();
    }
}

// z = (L U)^-1 r of a block, with its factor and schedules in global memory and
// only its vector y in LDS
__device__ inline void ilu_solve_block(const IluArgs &g, int32_t b, const double *__restrict__ r,
                                       double *__restrict__ z, double *y) {
    const int32_t r0 = b * g.B, r1 = min(g.n, r0 + g.B);
    const int tid = threadIdx.x;
    const double *__restrict__ v = g.fval;
    const uint16_t *__restrict__ col = g.fcol;
    // the block's right-hand side into LDS, all loads in flight at once
    for (int32_t i = tid; i < r1 - r0; i += kIluThreads) y[i] = r[g.rdev[r0 + i]];
    __syncthreads();
    // L y = r (unit diagonal), in place
    for (int32_t l = g.lvb_f[b]; l < g.lvb_f[b + 1]; ++l) {
        for (int32_t t = g.lptr_f[l] + tid; t < g.lptr_f[l + 1]; t += kIluThreads) {
            const int4 m = g.slot_f[t];
            double s = y[m.x];
            for (int32_t p = m.y; p < m.z; ++p) s -= v[p] * y[col[p]];
            y[m.x] = s;
        }
        __syncthreads();
    }
    // U z = y, in place
    for (int32_t l = g.lvb_b[b]; l < g.lvb_b[b + 1]; ++l) {
        for (int32_t t = g.lptr_b[l] + tid; t < g.lptr_b[l + 1]; t += kIluThreads) {
            const int4 m = g.slot_b[t];
            double s = y[m.x];
            for (int32_t p = m.y + 1; p < m.z; ++p) s -= v[p] * y[col[p]];
            y[m.x] = s / v[m.y];
        }
        __syncthreads();
    }
    for (int32_t i = tid; i < r1 - r0; i += kIluThreads) z[g.rdev[r0 + i]] = y[i];
}
__global__ __launch_bounds__(kIluThreads) void ilu_solve_kernel(IluArgs g, const double *__restrict__ r,
                                                                double *__restrict__ z, const PcgState *st) {
    if (st && st->done) return;
    extern __shared__ double lds[];
    ilu_solve_block(g, blockIdx.x, r, z, lds);
}

// One substitution over a block staged in LDS: level by level, one lane per row,
// the row's entries in their order.  A level holds few rows (2 or 3 for blocks
// of 128 unknowns), so its time is the chain y -> sum -> y: the slots of the
// level after next and the first kIluAhead entries of the next level, which do
// not depend on y, are read ahead.  Rows past the wavefront's 64 of a level take
// the same steps unhurried.  (Eight lanes per row with their sums combined by a
// tree took 30 us, inverted triangles of 16 rows 14, but a BiCGStab solve to
// 1e-12 carries their other rounding to 1e-9 of a face flux: the sums keep the
// order of ilu_solve_kernel, and the quotient is the correctly rounded one, by
// Markstein's theorem from the correctly rounded reciprocal, with one more
// correction so that the second starts within an ulp.  The theorem wants a
// reciprocal, a quotient and a remainder that neither overflow nor lose bits
// below the smallest normal number: numerators and pivots from 2^-500 to 2^500,
// and zero numerators.  A block with another one is solved again with divisions:
// asked row by row the question took 5 of 43 us.)
constexpr int kIluAhead = 8;
__device__ inline bool ilu_middle(double a) {  // 2^-500 <= |a| < 2^501
    return ((uint32_t)((uint64_t)__double_as_longlong(a) >> 52) & 0x7ffu) - 523u <= 1000u;
}
struct IluRow {
    ushort4 m;  // local row, its entries [y, z); w = 0: no row
    double v[kIluAhead], d, di;
    uint16_t c[kIluAhead];
    bool wide;  // of the wavefront's rows: more than kIluAhead / 2 entries
};
// zero: the place of a 0 in y.  True where a lane met a numerator that the
// quotients are not made for.
template <bool BACK>
__device__ inline bool ilu_sweep(int nlev, const uint16_t *__restrict__ lp, const ushort4 *__restrict__ slot,
                                 const double *__restrict__ val, const uint16_t *__restrict__ col,
                                 const double *__restrict__ dinv, double *y, uint16_t zero) {
    const int lane = threadIdx.x;
    bool off = false;
    const ushort4 none = make_ushort4(0, 0, 0, 0);
    auto get = [&](int t, int t1) { return t < t1 ? slot[t] : none; };
    constexpr int H = kIluAhead / 2;  // rows of more entries take a second turn of loads
    auto load = [&](IluRow &R, const ushort4 &m) {
        R.m = m;
        auto entry = [&](int k) {  // past the row: 0 times 0
            const bool on = m.y + k < m.z;
            const int p = on ? m.y + k : 0;
            const double v = val[p];
            const uint16_t c = col[p];
            R.v[k] = on ? v : 0.0;
            R.c[k] = on ? c : zero;
        };
#pragma unroll
        for (int k = 0; k < H; ++k) entry(k);
        R.wide = __any(m.y + H < m.z);
        if (R.wide)
#pragma unroll
            for (int k = H; k < kIluAhead; ++k) entry(k);
        R.d = BACK && m.w ? val[m.y - 1] : 1.0;
        R.di = BACK ? dinv[m.x] : 1.0;
    };
    // the row's sum and store; between its reads of y and their use the loads of `next`
    auto run = [&](const IluRow &R, IluRow *next, const ushort4 &mn) {
        double s = y[R.m.x], x[kIluAhead];
#pragma unroll
        for (int k = 0; k < H; ++k) x[k] = y[R.c[k]];
        if (R.wide)
#pragma unroll
            for (int k = H; k < kIluAhead; ++k) x[k] = y[R.c[k]];
        if (next) load(*next, mn);
#pragma unroll
        for (int k = 0; k < H; ++k) s = fma(-R.v[k], x[k], s);
        if (R.wide) {
#pragma unroll
            for (int k = H; k < kIluAhead; ++k) s = fma(-R.v[k], x[k], s);
            for (int p = R.m.y + kIluAhead; p < R.m.z; ++p) s = fma(-val[p], y[col[p]], s);
        }
        if (BACK) {
            double q = s * R.di;
            q = fma(fma(-R.d, q, s), R.di, q);
            off |= R.m.w && !(ilu_middle(s) || __double_as_longlong(s) == 0);
            s = fma(fma(-R.d, q, s), R.di, q);
        }
        if (R.m.w) y[R.m.x] = s;
    };
    auto at = [&](int l) { return (int)lp[min(l, nlev + 1)]; };  // lp is padded by copies of its end
    int t0 = lp[0], t1 = lp[1], t2 = at(2), t3 = at(3);
    ushort4 m1 = get(t1 + lane, t2);
    IluRow R0;
    load(R0, get(t0 + lane, t1));
    for (int l = 0; l < nlev; ++l) {
        const int t4 = at(l + 4);
        const ushort4 m2 = get(t2 + lane, t3);
        IluRow R1;
        run(R0, &R1, m1);
        for (int t = t0 + kIluThreads; t < t1; t += kIluThreads) {  // the same trip count in every lane
            IluRow R;
            load(R, get(t + lane, t1));
            run(R, nullptr, none);
        }
        // one wavefront, whose LDS accesses are in order: nothing to wait for
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        t0 = t1;
        t1 = t2;
        t2 = t3;
        t3 = t4;
        R0 = R1;
        m1 = m2;
    }
    __syncthreads();
    return off;
}
static_assert(kIluThreads == 64, "a substitution is one wavefront's");

// z = (L U)^-1 r of a block, one wavefront.  The block's values, columns,
// schedules and vector are staged in LDS by coalesced loads, all in flight
// together; the substitutions then touch LDS only.  (Reading slots and entries
// from global memory level by level cost two dependent round trips per level,
// ~0.57 us: 67 us per application at 113 k unknowns in blocks of 128, 43 us
// staged.  What bounds it is still the chain of levels, ~0.3 us each: reads of
// slots, entries and y in turn; a third stage of the pipeline did not shorten
// it.)
__global__ __launch_bounds__(kIluThreads) void ilu_solve_lds_kernel(IluArgs g, IluLds L, const double *__restrict__ r,
                                                                    double *__restrict__ z, const PcgState *st) {
    if (st && st->done) return;
    extern __shared__ double lds[];
    double *y = lds, *dinv = y + L.rows + 1, *val = dinv + L.rows;
    ushort4 *slf = reinterpret_cast<ushort4 *>(val + L.ents), *slb = slf + L.rows;
    uint16_t *lpf = reinterpret_cast<uint16_t *>(slb + L.rows), *lpb = lpf + L.levs + 3, *col = lpb + L.levs + 3;
    const int32_t b = blockIdx.x, r0 = b * g.B, nr = min(g.n, r0 + g.B) - r0;
    const int32_t e0 = g.fptr[r0], ne = g.fptr[r0 + nr] - e0;
    const int32_t f0 = g.lvb_f[b], nf = g.lvb_f[b + 1] - f0, b0 = g.lvb_b[b], nb = g.lvb_b[b + 1] - b0;
    const int tid = threadIdx.x;
    bool off = false;
#pragma unroll 4
    for (int e = tid; e < ne; e += kIluThreads) {
        val[e] = g.fval[e0 + e];
        col[e] = g.fcol[e0 + e];
    }
#pragma unroll 2
    for (int i = tid; i < nr; i += kIluThreads) {
        y[i] = r[g.rdev[r0 + i]];
        const double d = g.fval[g.fdiag[r0 + i]];
        dinv[i] = 1.0 / d;
        off |= !ilu_middle(d);
        const int4 mf = g.slot_f[r0 + i], mb = g.slot_b[r0 + i];
        slf[i] = make_ushort4((uint16_t)mf.x, (uint16_t)(mf.y - e0), (uint16_t)(mf.z - e0), 1);
        slb[i] = make_ushort4((uint16_t)mb.x, (uint16_t)(mb.y + 1 - e0), (uint16_t)(mb.z - e0), 1);
    }
    if (tid == 0) y[L.rows] = 0.0;
    // level pointers, the end repeated (the sweeps look up to four levels ahead, at most at entry nlev + 1)
    for (int l = tid; l < nf + 3; l += kIluThreads) lpf[l] = (uint16_t)((l < nf ? g.lptr_f[f0 + l] : r0 + nr) - r0);
    for (int l = tid; l < nb + 3; l += kIluThreads) lpb[l] = (uint16_t)((l < nb ? g.lptr_b[b0 + l] : r0 + nr) - r0);
    __syncthreads();
    const uint16_t zero = (uint16_t)L.rows;
    ilu_sweep<false>(nf, lpf, slf, val, col, nullptr, y, zero);  // L y = r (unit diagonal), in place
    off |= ilu_sweep<true>(nb, lpb, slb, val, col, dinv, y, zero);  // U z = y, in place
    if (__any(off)) {
        ilu_solve_block(g, b, r, z, y);
        return;
    }
    for (int i = tid; i < nr; i += kIluThreads) z[g.rdev[r0 + i]] = y[i];
}

void Ilu::factor(hipStream_t s, const double *A, int *bad) {
    if (a_.nblk == 0) return;
    hipLaunchKernelGGL(ilu_factor_kernel, dim3(a_.nblk), dim3(kIluThreads), 0, s, a_, A, bad);
    VAG_HIP(hipGetLastError());
}

void Ilu::apply(hipStream_t s, const double *r, double *z, const PcgState *st) const {
    if (a_.nblk == 0) return;
    if (in_lds_) {
        hipLaunchKernelGGL(ilu_solve_lds_kernel, dim3(a_.nblk), dim3(kIluThreads), lds_.bytes(), s, a_, lds_, r, z, st);
        VAG_HIP(hipGetLastError());
        return;
    }
    const size_t lds = (size_t)std::min(a_.B, a_.n) * sizeof(double);
    hipLaunchKernelGGL(ilu_solve_kernel, dim3(a_.nblk), dim3(kIluThreads), lds, s, a_, r, z, st);
    VAG_HIP(hipGetLastError());
}

}  // namespace vag
