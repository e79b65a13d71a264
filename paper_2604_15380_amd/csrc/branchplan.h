// How the wide branch layers' scratch is cut (host code without HIP).
//
// Atoms go through the branches in ranges, each with its own Y (and, blended
// with forces, dE_h/dY) in the scratch, and a range's tiles in chunks with
// their own activations.  Where memory is free there is one range: Y's row is
// wider than the buffers whose space it takes for shared layers much wider than
// F (1,024 in FP32: 6 KiB an atom against 2.3 + the basis rows at F = 64), and
// blended dE_h/dY is heads times as much (256 KiB an atom at 64 heads).
#pragma once

#include <stddef.h>

struct BranchPlan {
  size_t y_row, dyh_row, tile;   // bytes per atom of Y and dE_h/dY, and of a tile
  int TM;                        // rows of a tile
  long long tiles;               // most tiles of all atoms
};

// Bytes that a range's rows, and the tiles beside them, are given at most
// where memory is allocated freely.
constexpr size_t BRANCH_SCRATCH_TARGET = (size_t)1 << 30;

// bytes of the rows of a range of n atoms
inline size_t branch_range_bytes(const BranchPlan& p, size_t n) {
  return ((n * p.y_row + 255) & ~(size_t)255) + ((n * p.dyh_row + 255) & ~(size_t)255);
}

// scratch that the branches of N atoms cannot do without
inline size_t branch_scratch_min(const BranchPlan& p, int N) {
  return branch_range_bytes(p, N < p.TM ? N : p.TM) + p.tile;
}

// scratch that takes them at once, as far as BRANCH_SCRATCH_TARGET goes
inline size_t branch_scratch_full(const BranchPlan& p, int N) {
  size_t rows = branch_range_bytes(p, N), all = (size_t)p.tiles * p.tile;
  if (rows > BRANCH_SCRATCH_TARGET) rows = BRANCH_SCRATCH_TARGET;
  if (all > BRANCH_SCRATCH_TARGET) all = BRANCH_SCRATCH_TARGET;
  const size_t full = rows + all, least = branch_scratch_min(p, N);
  return full > least ? full : least;
}

// Atoms of a range (the last may have fewer) with `scratch` bytes, at least
// branch_scratch_min: all where their rows take at most half of it, or all
// tiles fit beside them; else as many, in equal ranges, as take half.
inline int branch_range(const BranchPlan& p, int N, size_t scratch) {
  const size_t rows = branch_range_bytes(p, N);
  if (rows + p.tile <= scratch && (rows <= scratch / 2 || rows + (size_t)p.tiles * p.tile <= scratch)) return N;
  const size_t least = N < p.TM ? N : p.TM;
  size_t n = scratch / 2 > 512 ? (scratch / 2 - 512) / (p.y_row + p.dyh_row) : 0;
  if (n < least || branch_range_bytes(p, n) + p.tile > scratch) n = least;
  const size_t k = ((size_t)N + n - 1) / n;
  return (int)(((size_t)N + k - 1) / k);
}
