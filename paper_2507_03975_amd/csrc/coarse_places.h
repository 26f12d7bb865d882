// coarse_places.h -- places (in values) of a multigrid level's operator in its
// piece of memory, and of what the one-workgroup kernels load of it. Plain
// constexpr arithmetic, so that a host program can go through every load.
//
// The piece holds diag, ay, ax of n cells each and ends on 32 values. The
// kernels load two neighbouring values at a time for the cells (l, l + 1), l
// even. Two of these loads reach one value past their array: that of l = n - 1
// (n odd: the piece has room behind it) and the couplings south of a pair
// across the first row's end (nx odd, n possibly a multiple of 32): they come
// from ay, so ay is not the last array.
#pragma once

namespace gsis {

constexpr int kPieceValues = 32;
constexpr int op_ay(int n) { return n; }
constexpr int op_ax(int n) { return 2 * n; }
// from a cell's place to the coupling south of it in ay and west of it in ax;
// at the south and west edges those stored (as zeros) for the last row and for
// the row's end
constexpr int south_step(int j, int nx, int n) { return j > 0 ? -nx : n - nx; }
constexpr int west_step(int i, int nx) { return i > 0 ? -1 : nx - 1; }

}  // namespace gsis
