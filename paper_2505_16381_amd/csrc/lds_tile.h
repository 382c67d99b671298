// Layout of the chunk-transform adjoint's tiles in LDS (plain C++: the test of it compiles it alone): rows of W 16-bit elements, no
// padding.  The sixteen-byte pieces of a row -- sixteen at W = 128; eight, two rows to a turn of the banks, at W = 64 -- are permuted by an
// exclusive or with a number made of the row, such that neither sixteen rows' pieces of the same columns, which a fragment with the contraction along
// the row takes, nor four rows' 64 bytes, which a transposing read takes, fall on the same banks.  (A padded row serves the former
// alone.)
#pragma once

#ifndef XCD_FN
#ifdef __HIP__
#define XCD_FN __host__ __device__ inline
#else
#define XCD_FN inline
#endif
#endif

namespace path {

template <int W> struct TurnedTile {
    static_assert(W == 64 || W == 128, "rows of sixteen or eight pieces");
    static XCD_FN int turn(int row) { return W == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : ((row & 2) << 1) | ((row >> 2) & 3); }
    static XCD_FN int at(int row, int col) { return row * W + ((((col >> 3) ^ turn(row)) << 3) | (col & 7)); }
};

// The lane's share of such addresses, in bytes, so that what is left per access is an immediate offset or one exclusive or with a constant
// (tiles start on multiples of 256 bytes, blocks on multiples of 32 rows and columns; l32 = lane % 32, h = lane / 32):
//   nat   row l32, eight columns from 8 h on          (column + c, c a multiple of 16: xor 2 c; row + r, r a multiple of 32: + 2 W r)
//   tr    row 8 h + (l32 % 16) / 4, the lane's four columns of a transposing read      (column + c, c a multiple of 32: xor 2 c; row + 16 s: + 32 W s; row + 4: xor 16, + 8 W)
//   vec   row l32, four columns from 4 h on           (column + c, c a multiple of 8: xor 2 c)
//   elem  row 4 h, column l32                         (column + c, c a multiple of 32: xor 2 c; row + 8 q + r: xor (q % 2) << 5, xor r << 6 or, at W = 64, r / 2 << 6, + 2 W (8 q + r))
//   copy  eight columns of thread tid's piece of a copy by whole rows      (piece + 512 u: + 8192 u)
template <int W> struct TurnedLane {
    typedef TurnedTile<W> L;
    unsigned nat, tr, vec, elem, copy;
    XCD_FN TurnedLane(int tid) {
        const int l32 = tid & 31, h = (tid >> 5) & 1, j = l32 & 15;
        nat = 2 * L::at(l32, 8 * h);
        tr = 2 * L::at(8 * h + (j >> 2), (l32 & 16) + 4 * (j & 3));
        vec = 2 * L::at(l32, 4 * h);
        elem = 2 * L::at(4 * h, l32);
        copy = 2 * L::at(tid / (W / 8), (tid % (W / 8)) * 8);
    }
    XCD_FN unsigned nat_at(int row, int col) const { return 2 * W * row + (nat ^ (2 * col)); }
    XCD_FN unsigned tr_at(int row, int col, int four) const { return 2 * W * (row + 4 * four) + (tr ^ (2 * col) ^ (16 * four)); }
    XCD_FN unsigned vec_at(int row, int col) const { return 2 * W * row + (vec ^ (2 * col)); }
    // (two steps: the first once per block, the second with constants)
    XCD_FN unsigned elem_at(int row, int col) const { return 2 * W * row + (elem ^ (2 * col)); }
    static XCD_FN unsigned elem_step(unsigned a, int q, int r) { return (a ^ ((q & 1) << 5 | (W == 128 ? r : r >> 1) << 6)) + 2 * W * (8 * q + r); }
    XCD_FN unsigned copy_at(int u) const { return copy + 8192 * u; }
};

}  // namespace path
