// Several explicit steps per launch on small hexahedral meshes.  A step of a few
// thousand control volumes is one launch that waits for the last one, 3.6 us
// whatever it computes (transport.hip), so a call of many steps cuts the mesh
// into parts, one block each: a block loads the states of its rows and of all
// rows that these reach upstream within K steps, advances them K steps in LDS
// (step t computes the rows within K - t entries of its own, so nothing is
// exchanged) and stores its own rows.  Rows in several parts are computed in
// each of them.  Every row gets the additions of transport_step_kernel in its
// order, so the states are the same bits.
#include "reduce.h"

namespace vag {

// T row by row (kHaloWidth entries side by side; len: entries | the entries of
// transport_step_kernel's batches of four << 8) from the packed operator.
__global__ __launch_bounds__(kSliceRows) void halo_rows_kernel(UpwindOp T, HaloRows R, int *cut) {
    const int32_t sl = blockIdx.x;
    const int lane = threadIdx.x;
    const uint16_t m = T.meta[sl * kSliceRows + lane];
    const int32_t i = sl * kSliceRows + (m >> 8);
    const bool row = i < T.nrow;
    const int cnt = row ? (m & 255) : 0;
    const int width = __shfl(cnt, 0, 64);  // a slice's rows are sorted longest first
    if (width > kHaloWidth) {              // whole wavefronts
        if (lane == 0) atomicMax(cut, kHaloSteps);
        if (row) R.len[i] = 0;
        return;
    }
    const int64_t o = (int64_t)i * kHaloWidth;
    int64_t p = T.slice_ptr[sl] + lane;
    for (int k = 0; k < width; ++k) {
        const bool has = cnt > k;
        const int n = __popcll(__ballot(has));
        if (has) {
            R.col[o + k] = T.tcol[p];
            R.val[o + k] = T.tval[p];
        }
        p += n;
    }
    if (row) R.len[i] = cnt | (width & ~3) << 8;
}

// The rows of part b: its share of the cells, the faces and nodes whose first
// cell it has, then level by level the rows that the last level's entries name
// (row nrow, the constant control volume, is everybody's).  cut: the steps by
// which kHaloSteps has to be reduced for every part to fit.
__global__ __launch_bounds__(1024) void halo_grow_kernel(int32_t nc, int32_t nf, int32_t nn,
                                                         const int32_t *__restrict__ frac_cell,
                                                         const int32_t *__restrict__ ncp,
                                                         const int32_t *__restrict__ ncl, HaloRows R, HaloParts H,
                                                         int *cut) {
    __shared__ unsigned seen[kHaloMaxRows / 32];
    __shared__ int32_t list[kHaloRows];
    __shared__ int n;
    const int tid = threadIdx.x, b = blockIdx.x;
    const int32_t nrow = nc + nf + nn;
    const int32_t lo = (int32_t)((int64_t)nc * b / H.nparts), hi = (int32_t)((int64_t)nc * (b + 1) / H.nparts);
    for (int k = tid; k < kHaloMaxRows / 32; k += 1024) seen[k] = 0;
    if (tid == 0) n = 0;
    __syncthreads();
    auto add = [&](int32_t i) {
        const unsigned bit = 1u << (i & 31);
        if (atomicOr(&seen[i >> 5], bit) & bit) return;
        const int s = atomicAdd(&n, 1);
        if (s < kHaloRows) list[s] = i;
    };
    for (int32_t i = lo + tid; i < hi; i += 1024) add(i);
    for (int32_t f = tid; f < nf; f += 1024) {
        const int32_t K = frac_cell[2 * f];
        if (K >= lo && K < hi) add(nc + f);
    }
    for (int32_t v = tid; v < nn; v += 1024) {
        const int32_t K = ncp[v] < ncp[v + 1] ? ncl[ncp[v]] >> 3 : 0;  // a node of no cell: the first part
        if (K >= lo && K < hi) add(nc + nf + v);
    }
    __syncthreads();
    int32_t *level = H.level + b * (kHaloSteps + 1);
    int from = 0, to = n, j = 0;
    if (tid == 0) level[0] = to;
    for (; to <= kHaloRows && j < kHaloSteps; ++j) {
        __syncthreads();  // everyone has read n
        for (int e = tid; e < 16 * (to - from); e += 1024) {
            const int32_t i = list[from + (e >> 4)];
            const int k = e & 15;
            if (k < (R.len[i] & 255)) {
                const int32_t c = R.col[(int64_t)i * kHaloWidth + k];
                if (c < nrow) add(c);
            }
        }
        __syncthreads();
        from = to;
        to = n;
        if (tid == 0) level[j + 1] = to;
    }
    // level j is the last one counted; it fits unless the loop ended for it
    const int steps = to <= kHaloRows ? j : j - 1;
    if (tid == 0 && steps < kHaloSteps) atomicMax(cut, kHaloSteps - max(steps, 0));
    for (int r = tid; r < min(to, kHaloRows); r += 1024) H.list[b * kHaloRows + r] = list[r];
}

// The parts' rows with local columns, entry by entry (a block's loads of a
// step's launch are then of consecutive addresses).
__global__ __launch_bounds__(1024) void halo_pack_kernel(int32_t nrow, const double *__restrict__ diag, HaloRows R,
                                                         HaloParts H, const int *__restrict__ cut) {
    extern __shared__ uint16_t slot[];  // [nrow]
    const int steps = kHaloSteps - *cut;
    if (steps < 1) return;
    const int tid = threadIdx.x, b = blockIdx.x;
    const int32_t *list = H.list + b * kHaloRows, *level = H.level + b * (kHaloSteps + 1);
    const int n = level[steps], m = level[steps - 1];
    for (int r = tid; r < n; r += 1024) slot[list[r]] = (uint16_t)r;
    __syncthreads();
    for (int r = tid; r < m; r += 1024) {
        const int32_t i = list[r], len = R.len[i];
        H.len[b * kHaloRows + r] = (uint16_t)len;
        H.diag[b * kHaloRows + r] = diag[i];
        const int64_t o = (int64_t)b * kHaloWidth * kHaloRows + r;
        for (int k = 0; k < (len & 255); ++k) {
            const int32_t c = R.col[(int64_t)i * kHaloWidth + k];
            H.col[o + k * kHaloRows] = c < nrow ? slot[c] : (uint16_t)kHaloRows;
            H.val[o + k * kHaloRows] = R.val[(int64_t)i * kHaloWidth + k];
        }
    }
}

// `steps` steps of the block's part: a launch's 3.3 us and about 1.5 us to load
// the part are shared by up to eight steps of 0.4 us (LDS gathers; the halo's
// rows grow with the steps, so more than eight gain little).  A thread keeps the operator's rows tid and
// tid + 1024 in registers; a step gathers from one copy of the states in LDS
// and writes the other.  Columns of rows that a step computes were computed by
// the step before (their level is at most one higher).
__global__ __launch_bounds__(1024) void transport_halo_kernel(int32_t nrow, int steps, HaloParts H,
                                                              const double *__restrict__ c_in,
                                                              double *__restrict__ c_out) {
#pragma clang fp contract(off)  // as transport_step_kernel adds
    constexpr int RT = kHaloRows / 1024;
    __shared__ double xs[2][kHaloRows + 1];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int32_t *level = H.level + b * (kHaloSteps + 1);
    const int n = level[steps], m = level[steps - 1];
    double d[RT], v[RT][kHaloWidth];
    int32_t row[RT];
    int cnt[RT], four[RT], width[RT];
    uint16_t c[RT][kHaloWidth];
#pragma unroll
    for (int u = 0; u < RT; ++u) {
        const int r = tid + 1024 * u;
        row[u] = r < n ? H.list[b * kHaloRows + r] : nrow;
        const int len = r < m ? H.len[b * kHaloRows + r] : 0;
        d[u] = r < m ? H.diag[b * kHaloRows + r] : 0.0;
        cnt[u] = len & 255;
        four[u] = len >> 8;
    }
#pragma unroll
    for (int u = 0; u < RT; ++u) {
        const int r = tid + 1024 * u;
        const int64_t o = (int64_t)b * kHaloWidth * kHaloRows + r;
#pragma unroll
        for (int k = 0; k < kHaloWidth; ++k) {
            const bool has = k < cnt[u];
            c[u][k] = has ? H.col[o + k * kHaloRows] : (uint16_t)kHaloRows;
            v[u][k] = has ? H.val[o + k * kHaloRows] : 0.0;
        }
        if (r < n) xs[0][r] = c_in[row[u]];
        width[u] = 0;
        for (int k = 0; k < kHaloWidth; k += 4)
            if (__any(k < cnt[u])) width[u] = k + 4;  // of the wavefront
    }
    if (tid == 0) xs[0][kHaloRows] = xs[1][kHaloRows] = c_in[nrow];
    __syncthreads();
    for (int t = 0; t < steps; ++t) {
        const double *x = xs[t & 1];
        double *y = xs[(t + 1) & 1];
        const int lim = level[steps - 1 - t];
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            const int r = tid + 1024 * u;
            if (r < lim) {
                double a0 = d[u] * x[r], a1 = 0.0, a2 = 0.0, a3 = 0.0;
#pragma unroll
                for (int k = 0; k < kHaloWidth; k += 4) {
                    if (k >= width[u]) break;
                    const double x0 = x[c[u][k]], x1 = x[c[u][k + 1]], x2 = x[c[u][k + 2]], x3 = x[c[u][k + 3]];
                    const double p0 = k < cnt[u] ? v[u][k] * x0 : 0.0;
                    const double p1 = k + 1 < cnt[u] ? v[u][k + 1] * x1 : 0.0;
                    const double p2 = k + 2 < cnt[u] ? v[u][k + 2] * x2 : 0.0;
                    const double p3 = k + 3 < cnt[u] ? v[u][k + 3] * x3 : 0.0;
                    const bool batch = k < four[u];  // past the slice's batches of four: one sum
                    a1 = a1 + p0;
                    a1 = batch ? a1 : ((a1 + p1) + p2) + p3;
                    a2 = batch ? a2 + p1 : a2;
                    a3 = batch ? a3 + p2 : a3;
                    a0 = batch ? a0 + p3 : a0;
                }
                y[r] = (a0 + a1) + (a2 + a3);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < RT; ++u)
        if (tid + 1024 * u < level[0]) c_out[row[u]] = xs[steps & 1][tid + 1024 * u];
}

void launch_halo_build(hipStream_t s, const UpwindOp &T, int32_t nc, int32_t nf, int32_t nn, const int32_t *frac_cell,
                       const int32_t *ncp, const int32_t *ncl, const HaloRows &R, const HaloParts &H, int *cut) {
    if (T.nrow != nc + nf + nn || T.nrow > kHaloMaxRows || H.nparts < 1)
        throw Error(VAG_ERR_ARG, "internal: halo of too many rows");
    hipLaunchKernelGGL(halo_rows_kernel, dim3((T.nrow + kSliceRows - 1) / kSliceRows), dim3(kSliceRows), 0, s, T, R,
                       cut);
    VAG_HIP(hipGetLastError());
    hipLaunchKernelGGL(halo_grow_kernel, dim3(H.nparts), dim3(1024), 0, s, nc, nf, nn, frac_cell, ncp, ncl, R, H, cut);
    VAG_HIP(hipGetLastError());
    const size_t lds = 2 * (size_t)T.nrow;
    VAG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(halo_pack_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kHaloMaxRows));
    hipLaunchKernelGGL(halo_pack_kernel, dim3(H.nparts), dim3(1024), lds, s, T.nrow, T.tdiag, R, H, cut);
    VAG_HIP(hipGetLastError());
}
void launch_transport_halo(hipStream_t s, int32_t nrow, int steps, const HaloParts &H, const double *c_in,
                           double *c_out) {
    if (steps < 1 || steps > kHaloSteps) throw Error(VAG_ERR_ARG, "internal: halo of too many steps");
    hipLaunchKernelGGL(transport_halo_kernel, dim3(H.nparts), dim3(1024), 0, s, nrow, steps, H, c_in, c_out);
    VAG_HIP(hipGetLastError());
}

}  // namespace vag
