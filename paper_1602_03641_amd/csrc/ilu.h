// Block-Jacobi ILU(0) preconditioner (the third preconditioner of the solver
// study in §5.3, where GMRES and BiCGStab use it with one block per MPI
// process).  Here a block is a run of `B` consecutive unknowns of the
// system's natural order (free nodes by node index, then kept fracture faces
// by face index), factored without fill in that order; the device rows are
// stored in another order (sorted by length inside windows), so every row
// carries its device row and its factor entries their position in the
// device matrix.
#pragma once

#include <algorithm>

#include "vag_internal.h"

namespace vag {

constexpr int kIluMaxBlock = 8192;  // rows per block: the solve keeps a block's vector in LDS
constexpr int kIluDefaultBlock = 128;

struct IluArgs {
    int32_t n, B, nblk;
    const int32_t *fptr;    // [n+1] factor entries of natural row o: [fptr[o], fptr[o+1])
    const uint16_t *fcol;   // local column (natural column - block start), ascending per row
    const int32_t *fsrc;    // position of the entry in the device matrix
    const int32_t *fdiag;   // [n] index of row o's diagonal entry
    const int32_t *rdev;    // [n] device row of natural row o
    // level schedules of the lower (forward) and upper (backward) dependency
    // graphs: block b's levels are [lvb[b], lvb[b+1]); level l's rows are
    // rows[lptr[l] .. lptr[l+1]) (natural indices, a permutation of the block)
    const int32_t *lvb_f, *lptr_f, *rows_f;
    const int32_t *lvb_b, *lptr_b, *rows_b;
    // per schedule slot, what the substitutions read in one 16-byte load:
    // forward {row - block start, first entry, diagonal entry, 0},
    // backward {row - block start, diagonal entry, end of the row, 0}
    const int4 *slot_f, *slot_b;
    double *fval;           // factor values: L below the diagonal (unit diagonal implied), U from it
};

// LDS of the solve that stages a block's factor and schedules there: the same
// layout for every block, sized for the largest counts of any block.
struct IluLds {
    int32_t rows = 0, ents = 0, levs = 0;  // rows, factor entries and levels (of either sweep) of a block
    size_t slots_f() const { return 8 * (size_t)(2 * rows + 1 + ents); }  // after y, 0, 1 / diag and the values
    size_t bytes() const { return slots_f() + 16 * (size_t)rows + 2 * (2 * (size_t)(levs + 3) + ents); }
    static constexpr size_t kMax = 160 * 1024;  // of a CU
    // entry and slot indices inside a block are 16-bit there
    bool fits() const { return rows > 0 && ents <= 65535 && bytes() <= kMax; }
    // Whether nblk such blocks are solved faster there.  Not where a level is a
    // row (blocks of at most a line of the mesh): the chain is as long, and there
    // is nothing to share the staging (an application in LDS / in global memory,
    // us: 48^3 cells, blocks of 64 rows in 47 levels, 44 / 49; of 48 in 47, 48 /
    // 41; 128^3, 64 in 64, 517 / 447; 200 x 200 x 1, 192 in 192, 301 / 138).  And
    // not where the blocks take turns because few fit on a CU, while the other
    // kernel, whose blocks need 8 bytes of LDS per row, has up to 32 there at once
    // (80^3, blocks of 512, 2 on a CU, 2.0 turns, 159 / 218; 96^3, 3.4 turns, 343 /
    // 305; 128^3, 8 turns, 983 / 512; with 10 on a CU, blocks of 192: 112^3, 3.2
    // turns, 372 / 359; 128^3, 4.3 turns, where the other kernel takes turns too,
    // 570 / 641).
    bool pays(int64_t nblk) const {
        if (!fits() || 4 * rows < 5 * levs) return false;
        constexpr int64_t cus = 256, most = 32;
        const int64_t per = std::min<int64_t>(most, kMax / bytes());  // on a CU
        return nblk <= 3 * cus * per || (per >= 6 && nblk > cus * most);
    }
};

class Ilu {
public:
    // Host symbolic phase from the device matrix's pattern (once per handle
    // and block size); uploads on the stream.
    void build(hipStream_t s, Tracker &tr, const Symbolic &S, int B);
    bool ready(int B) const { return B_ == B && a_.n > 0; }
    // Copies the device matrix values into the factor and factors every
    // block; *bad (device) receives 1 + the natural row of a zero or
    // non-finite pivot.
    void factor(hipStream_t s, const double *A, int *bad);
    // z = (L U)^-1 r block by block (device order vectors); skipped when
    // st && st->done.
    void apply(hipStream_t s, const double *r, double *z, const PcgState *st) const;
    int levels() const { return nlev_; }
    bool in_lds() const { return in_lds_; }  // the solve stages its blocks in LDS
    int64_t entries() const { return nent_; }

private:
    int B_ = 0, nlev_ = 0;
    int64_t nent_ = 0;
    IluArgs a_{};
    IluLds lds_;
    bool in_lds_ = false;  // lds_.pays
    DBuf<int32_t> fptr_, fsrc_, fdiag_, rdev_, lvb_f_, lptr_f_, rows_f_, lvb_b_, lptr_b_, rows_b_;
    DBuf<int4> slot_f_, slot_b_;
    DBuf<uint16_t> fcol_;
    DBuf<double> fval_;
};

}  // namespace vag
