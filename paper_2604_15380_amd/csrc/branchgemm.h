// Operand layout of the wide branch layers' matrix products, shared by the
// host packing and the kernels in branch.hip.
//
// Operands live in blocks of 16 rows x KB k-values, 64 lanes x 16 bytes = 1
// KiB per plane: lane l holds row l % 16 (weights in FP64: see branch_feature)
// and k = (KB / 4) (l / 16) + e, e < KB / 4.  Both operands of a 16x16 MFMA
// take exactly this form, so a block moves between memory, LDS and registers
// as whole 16-byte lanes.
//   BF16: one plane of bf16, KB = 32.
//   FP32: three planes of bf16, KB = 32.  x = hi + mid + lo with hi = x and
//     mid = x - hi rounded to bf16, lo = x - hi - mid: every difference is
//     exact and the three 8-bit significands cover the 24 bits, so the planes
//     hold x exactly from 2^-110 up; below, to 2^-133, the smallest bf16
//     subnormal (the matrix cores keep subnormals).  A product with a value
//     below 2^-110 is so off by at most 2^-133 times the other operand.  An
//     infinity or NaN is in the lo plane alone and acts as in FP32; two
//     infinities that meet give NaN.  Rounded, not cut off: with cut-off
//     planes mid and lo have the sign of x, and the products that branch.hip
//     leaves out (mid lo, lo mid, lo lo) shrank every sum by 6e-8 of itself
//     per layer, which the energies' sums over atoms do not average away;
//     rounded, they are 6e-9 of either sign.
//   FP64: one plane of double, KB = 8.
#pragma once

#include "internal.h"

inline __host__ __device__ int branch_planes(int prec) { return prec == PAINN_FP32 ? 3 : 1; }
inline __host__ __device__ int branch_kb(int prec) { return prec == PAINN_FP64 ? 8 : 32; }

// The feature that row m of a weight block's 16 holds.  An FP64 accumulator
// register i of lane l is output row 4 i + l / 16, an FP32 one 4 (l / 16) + i;
// the FP64 weights are permuted so that a lane's four results are four
// consecutive features in every precision.
inline __host__ __device__ int branch_feature(int prec, int m) {
  return prec == PAINN_FP64 ? 4 * (m % 4) + m / 4 : m;
}

// Bytes of a packed layer of dout x din (both padded to 32).
inline size_t branch_pack_bytes(int prec, int dout, int din) {
  return (size_t)(pad32(dout) / 16) * (pad32(din) / branch_kb(prec)) * branch_planes(prec) * 1024;
}

// Rows of a tile, and the operand row bytes of a width-w layer.
constexpr int BRANCH_TM = 128, BRANCH_TM_SMALL = 32;
inline size_t branch_row_bytes(int prec, int w) {
  return (size_t)pad32(w) * (prec == PAINN_FP64 ? 8 : 2 * branch_planes(prec));
}
