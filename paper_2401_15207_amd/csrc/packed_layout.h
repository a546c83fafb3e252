// Where the elements of a weight lie in its MFMA fragment-order copy: shared by the packers and gemm_pk_k (gemm.hip) and by the update
// that writes the copies itself (update_pack.hip).
#pragma once
#include "common.h"
#include "kernels.h"

namespace hift {
namespace {

// Position in the packed copy of the 32-row block s of B (half = blocks in half of B).
__device__ __forceinline__ int64_t pk_block_pos(int64_t s, int order, int64_t half) {
  if (order == PK_ORDER_HALVES) {
    if (s >= 2 * half) return s;  // no such block: N is a multiple of 256 in this order
    const int64_t h = s >= half ? 1 : 0, i = s - h * half;
    return (i >> 2) * 8 + (i & 3) * 2 + h;
  }
  if (order == PK_ORDER_PAIR64) {
    const int64_t q = s & 3;
    return (s & ~int64_t(3)) | (q == 1 ? 2 : q == 2 ? 1 : q);
  }
  return s;
}

// Row r of a 32-row block of B sits where row pi(r) would (bits 2 and 3 of the index exchanged).  acc = mfma(B
// fragment, A fragment, acc) leaves in lane l, element e the entry (A row l % 32, B row 8 (e / 4) + 4 (l / 32) + e % 4);
// with the rows fed in this order, element e belongs to column 16 (e / 8) + 8 (l / 32) + e % 8 of the block: elements
// 0..7 and 8..15 are eight consecutive columns each, 16 bytes of a bf16 output row, and the epilogues of the
// packed-operand kernel write rows straight from the registers.
__device__ __forceinline__ int pi_row(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

// Product of eight bf16 pairs, each rounded once.
__device__ __forceinline__ hift_u32x4 scale8(hift_u32x4 a, hift_u32x4 b) {
  typedef __attribute__((ext_vector_type(8))) __bf16 v8bf;
  v8bf x = __builtin_bit_cast(v8bf, a);
  const v8bf y = __builtin_bit_cast(v8bf, b);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = static_cast<__bf16>(static_cast<float>(x[e]) * static_cast<float>(y[e]));
  return __builtin_bit_cast(hift_u32x4, x);
}

}  // namespace
}  // namespace hift
