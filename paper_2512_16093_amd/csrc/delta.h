// delta[bh][row] = dO[row] . O^s[row] from a saved O^s (rows beyond N: 0); one wavefront per 8 rows.
// The saved state's header must name this problem (shape, query block size, critical blocks per row): a
// buffer that no training forward pass of the same problem filled gives delta = lse = NaN, and with them NaN in
// every gradient, instead of plausible wrong numbers (the host cannot look without synchronising).
#pragma once
#include "common.h"

namespace sla {

__device__ __forceinline__ void delta_block(const DeltaArgs& X, int blk) {
  const long long gr = (long long)blk * 32 + (threadIdx.x >> 3);  // padded row index over all heads
  if (gr >= (long long)X.BH * X.rows_padded) return;
  const SavedHeader got = *X.hdr;
  const bool mine = got.magic == X.want.magic && got.B == X.want.B && got.H == X.want.H && got.N == X.want.N &&
                    got.block_q == X.want.block_q && got.n_c == X.want.n_c;
  const int bh = (int)(gr / X.rows_padded), row = (int)(gr - (long long)bh * X.rows_padded), part = threadIdx.x & 7;
  float s = 0.f;
  if (row < X.N) {
    const size_t off = ((size_t)bh * X.N + row) * D + 16 * part;   // (O^s: the library's own tensor)
    const int b_ = bh / X.H, h_ = bh - b_ * X.H;
    const bf16_t* drow = X.dout + b_ * X.ld.sb + h_ * X.ld.sh + (long long)row * X.ld.sn + 16 * part;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint4 a = *(const uint4*)(drow + 8 * h), b = *(const uint4*)(X.os + off + 8 * h);
      s += bf16_lo(a.x) * bf16_lo(b.x) + bf16_hi(a.x) * bf16_hi(b.x) + bf16_lo(a.y) * bf16_lo(b.y) + bf16_hi(a.y) * bf16_hi(b.y) +
           bf16_lo(a.z) * bf16_lo(b.z) + bf16_hi(a.z) * bf16_hi(b.z) + bf16_lo(a.w) * bf16_lo(b.w) + bf16_hi(a.w) * bf16_hi(b.w);
    }
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  s += __shfl_xor(s, 4);
  if (part == 0) {  // (the log-sum-exp goes to the workspace copy the other kernels read: poisoned alike)
    X.delta[gr] = mine ? s : __builtin_nanf("");
    X.lse2[gr] = mine ? X.lse_saved[gr] : __builtin_nanf("");
  }
}

}  // namespace sla
