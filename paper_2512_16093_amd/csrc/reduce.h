// Partial sums of dW and db (bwd_lin_q_kernel's), added up by workgroups in front of the launch that follows.
#pragma once
#include "common.h"

namespace sla {

// dW[x] and db[x] = sum over p of part[p][x] in a fixed order.  Workgroups 0 .. 255 take 64 entries of dW each (dw
// given), the last two 64 of db: 16 threads of four adjacent entries, 16 threads along p (every 16th partial, in four
// sums), joined pairwise in LDS (one after the other, the largest sums were rounded 15 times over: db of 4 x 4617 tokens
// off by 8.2e-8, now 5.9e-8).  Bound by reading the partials; with one thread per entry a chain of additions as long
// as the list bound it (768 partials of 64 KiB, dW and db: 141 us in two launches, now 256 partials and 5 us).
constexpr int RED_ENTRIES = 64;
inline int reduce_blocks(const ReduceArgs& R) { return (R.dw ? D * D / RED_ENTRIES : 0) + (R.db ? D / RED_ENTRIES : 0); }
__device__ __forceinline__ void reduce_block(const ReduceArgs& R, int blk, float4 (*red)[16]) {   // (red: shared, 16 rows)
  const float *dw_part = R.dw_part, *db_part = R.db_part;
  float *dw = R.dw, *db = R.db;
  const int n_part = R.n_part, dw_blocks = dw ? D * D / RED_ENTRIES : 0, t = threadIdx.x, col = t & 15, row = t >> 4;
  if (blk >= dw_blocks + (db ? D / RED_ENTRIES : 0)) return;
  const bool is_db = blk >= dw_blocks;
  const int n = is_db ? D : D * D, x = (is_db ? blk - dw_blocks : blk) * RED_ENTRIES + 4 * col;
  const float* part = (is_db ? db_part : dw_part) + x;
  auto add = [](float4& a, const float4& b) __attribute__((always_inline)) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; };
  float4 s[4] = {};
  int p = row;
  for (; p + 48 < n_part; p += 64)
#pragma unroll
    for (int u = 0; u < 4; ++u) add(s[u], *(const float4*)(part + (size_t)(p + 16 * u) * n));
  for (; p < n_part; p += 16) add(s[0], *(const float4*)(part + (size_t)p * n));
  add(s[0], s[1]);
  add(s[2], s[3]);
  add(s[0], s[2]);
  red[row][col] = s[0];
  __syncthreads();
  if (t < 16) {
    float4 v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = red[r][t];
#pragma unroll
    for (int step = 1; step < 16; step *= 2)
#pragma unroll
      for (int r = 0; r < 16; r += 2 * step) add(v[r], v[r + step]);
    *(float4*)((is_db ? db : dw) + x) = v[0];
  }
}

}  // namespace sla
