// wave_steps.h -- the steps of a wavefront recurrence that one wave runs, and
// the entries of the diagonal table it reads for them. Plain constexpr
// arithmetic: the kernels use it, and a host program can go through every
// wave of a launch with it.
//
// A workgroup's wave w owns rows 64 w to 64 w + 63 of the pass (or part) and
// runs step s at time s + w lag, in blocks of lag steps. Of the workgroup's
// waves the first nw hold rows. A block's loads are those of the steps one
// block later.
#pragma once

namespace gsis {

// entries of the diagonal table before the first and after the last diagonal
constexpr int kDiagPad = 256;

// First step of the first block a wave runs: the block that loads for its
// first active step. A wave without rows runs none (wave_last_step); it takes
// the first block of all, whose table entries exist whatever the grid.
constexpr int wave_first_step(int wave, int nw, int lag) {
  return wave < nw ? (wave * 64 / lag - 1) * lag : -lag;
}
// A wave runs the blocks that start at or before this step: its last lane's
// last column (before every block for a wave without rows; tend: the time
// after the workgroup's last block).
constexpr int wave_last_step(int wave, int nw, int nx, int tend, int lag) {
  return wave < nw ? nx + wave * 64 + 62 : -tend - lag;
}
// Diagonal of load l (l < lag) issued in the block that starts at step sb:
// upwards from row y0, and downwards (the reversed sweep) from reversed row r0.
constexpr int diag_up(int y0, int sb, int lag, int l) { return y0 + sb + lag + l; }
constexpr int diag_down(int nx, int ny, int r0, int sb, int lag, int l) {
  return nx + ny - 2 - (r0 + sb + lag + l);
}

}  // namespace gsis
