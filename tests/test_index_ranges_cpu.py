"""Entries of tables that kernels read by computed place: the arithmetic that
the kernels use (headers of plain constexpr functions), run on the host over
every wave or thread of a launch. No GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2507_03975_amd", "csrc")


def _run(tmp_path, name, text):
    src, exe = tmp_path / (name + ".cpp"), tmp_path / name
    src.write_text(text)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


DIAGONALS = r"""
#include <algorithm>
#include <cstdio>
#include "wave_steps.h"
using namespace gsis;
static long long reads = 0, bad = 0;
static void read(int nx, int ny, int rows_pp, int y0, int wave, int d, const char *what) {
  ++reads;
  if (d >= -kDiagPad && d < nx + ny - 1 + kDiagPad) return;
  if (++bad <= 20)
    printf("%s %d x %d, %d rows a pass, first row %d, wave %d: diagonal %d\n", what, nx, ny,
           rows_pp, y0, wave, d);
}
// one pass (or part) of rows_pp / 64 waves from row y0 on: every wave
static void pass(int nx, int ny, int rows_pp, int y0, int lag, bool down) {
  const int rows = std::min(rows_pp, ny - y0), nw = (rows + 63) / 64;
  const int tend = (nx + rows - 1 + (nw - 1) * lag + lag - 1) / lag * lag;
  for (int wave = 0; wave < rows_pp / 64; ++wave) {
    const int first = wave_first_step(wave, nw, lag), last = wave_last_step(wave, nw, nx, tend, lag);
    auto block = [&](int sb) {       // both ends of the block's lanes
      for (int l : {0, lag - 1})
        read(nx, ny, rows_pp, y0, wave,
             down ? diag_down(nx, ny, y0, sb, lag, l) : diag_up(y0, sb, lag, l),
             down ? "down" : "up");
    };
    block(first);
    int tb = -lag, blocks = 0;
    for (; tb < tend && tb - wave * lag < first; tb += lag) ++blocks;
    for (; tb < tend && tb - wave * lag <= last; tb += lag, ++blocks) block(tb - wave * lag + lag);
    for (; tb < tend; tb += lag) ++blocks;
    if (blocks != tend / lag + 1) { ++bad; printf("barriers\n"); }   // alike in every wave
  }
}
int main() {
  const int sizes[] = {1, 2, 3, 24, 31, 63, 64, 65, 100, 127, 128, 129, 200, 255, 256, 257, 383,
                       385, 449, 511, 512, 513, 577, 769, 1023, 1024, 1025, 2049, 4096, 4097};
  for (int nx : sizes)
    for (int ny : sizes)
      for (int rows_pp = 64; rows_pp <= 1024; rows_pp += 64)
        for (int y0 = 0; y0 < ny; y0 += rows_pp) {
          pass(nx, ny, rows_pp, y0, 8, false);
          pass(nx, ny, rows_pp, y0, 8, true);
          if (rows_pp <= 256) pass(nx, ny, rows_pp, y0, 12, true);
        }
  printf("%lld reads, %lld out of range\n", reads, bad);
  return bad != 0;
}
"""


def test_recurrence_diagonals(tmp_path):
    """The recurrence and the adjoint's reversed sweep: every wave of every
    pass or part, also those that hold no rows (a workgroup as large as a
    batch's largest problem, the last pass of a tall grid), reads entries of
    the diagonal table only."""
    _run(tmp_path, "diagonals", DIAGONALS)


OPERATOR = r"""
#include <cstdio>
#include "coarse_places.h"
using namespace gsis;
static long long reads = 0, bad = 0;
int main() {
  for (int nx = 1; nx <= 4096; ++nx)
    for (int ny = 1; nx * ny <= 4096; ++ny) {
      const int n = nx * ny, piece = (3 * n + kPieceValues - 1) / kPieceValues * kPieceValues;
      auto load = [&](int at, int values, const char *what) {
        ++reads;
        if (at >= 0 && at + values <= piece) return;
        if (++bad <= 20) printf("%d x %d, %s: values %d..%d of %d\n", nx, ny, what, at,
                                at + values - 1, piece);
      };
      for (int l = 0; l < n; l += 2) {
        const int i = l % nx, j = l / nx;
        load(l, 2, "diag");
        load(op_ax(n) + l, 2, "ax");
        load(op_ay(n) + l, 2, "ay");
        load(op_ay(n) + l + south_step(j, nx, n), 2, "ay, south");
        load(op_ax(n) + l + west_step(i, nx), 1, "ax, west");
      }
    }
  printf("%lld loads, %lld out of range\n", reads, bad);
  return bad != 0;
}
"""


def test_coarse_operator_pairs(tmp_path):
    """The one-workgroup multigrid cycle loads a level's operator two values
    at a time, up to one past the end of its arrays: never past the piece of
    memory that holds them, on every grid it can own."""
    _run(tmp_path, "operator", OPERATOR)
