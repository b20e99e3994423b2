// Block pooling / statistics, pooled scores and the three-way block selection.
//
// Steps 1-2 of the path: per-block channel means of Q and K, the score
// s[i][j] = mean(Q_i).mean(K_j)/sqrt(d), and per query block the n_c best key
// blocks (critical), the next n_m (marginal), the rest negligible, equal scores
// ranking by ascending j (Section 2.1 fixes only the Top-K ratio; the rest is
// this library's stated reading, see sla.h).  The same pass over Q, K, V also
// produces what the low-bit branch needs later: the per-query-block INT8 scale,
// the channel mean of K (K-smoothing) and the per-channel max |V| (FP8 scale).
#include "classify.h"

namespace sla {

// ---------------------------------------------------------------------------
// pool_stats: one workgroup per (tensor, b,h, 128-token group); 256 threads; thread
// (rg = t/16, cg = t%16) reads 8 channels of rows rg + 16 r, r = 0..7.
// HBM-bound: reads Q, K, V exactly once (6 N d bytes per slice), Q's workgroups first, then K's, then V's (which the
// 16-bit forward, the backward pass and the classification alone leave out: parts = 2).  A workgroup per tensor and
// not one for all three: a third of the loads, shared memory and reduction steps one behind another, which is what the
// smallest calls wait for, and three times the workgroups in flight (2 x 1024 tokens 8.2 -> 5.8 us, 24 x 4617 24 -> 17,
// 12 x 32760 78 -> 66, 40 x 75600 525 -> 500; Q and K alone 4 x 2187 7.3 -> 3.6, 12 x 32760 44 -> 35).
// The maxima of V leave as one row per workgroup, which finalize_block reduces: nothing has to be cleared
// beforehand and there are no atomics (the clearing launch alone was 1.4 us of the smallest calls' 61).
// ---------------------------------------------------------------------------
struct PoolArgs {
  const bf16_t *x[3];   // q, k, v
  Layout l[3];
  int N, block_q, Tq, Tk, groups, H, per_part;   // per_part: workgroups per tensor, BH * groups
  float *qbar, *kbar, *dq, *vmax_part;
  int8_t* q8;
};
__global__ void __launch_bounds__(256) pool_stats_kernel(const PoolArgs A) {
  __shared__ __attribute__((aligned(16))) float sums[16][2][D];
  __shared__ float s_amax[2][4], s_qmax[2];
  const int part = blockIdx.x / A.per_part, blk = blockIdx.x - part * A.per_part;
  const int bh = blk / A.groups, g = blk - bh * A.groups, N = A.N;
  const int t = threadIdx.x, cg = t & 15, rg = t >> 4;
  const int b_ = bh / A.H, h_ = bh - b_ * A.H;
  const Layout L = part == 0 ? A.l[0] : part == 1 ? A.l[1] : A.l[2];
  const bf16_t* src = (part == 0 ? A.x[0] : part == 1 ? A.x[1] : A.x[2]) + b_ * L.sb + h_ * L.sh + cg * 8;
  const int row0 = g * 128;
  uint4 x[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {  // (all eight in flight: rows past the end are read as the last one and dropped)
    const int row = row0 + rg + 16 * r;
    x[r] = *(const uint4*)(src + min(row, N - 1) * L.sn);
    if (row >= N) x[r] = make_uint4(0u, 0u, 0u, 0u);
  }
  float s[2][8] = {}, amax[2] = {0.f, 0.f};
  if (part == 2) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t w[4] = {x[r].x, x[r].y, x[r].z, x[r].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[0][2 * e] = fmaxf(s[0][2 * e], fabsf(bf16_lo(w[e])));
        s[0][2 * e + 1] = fmaxf(s[0][2 * e + 1], fabsf(bf16_hi(w[e])));
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t w[4] = {x[r].x, x[r].y, x[r].z, x[r].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = bf16_lo(w[e]), hi = bf16_hi(w[e]);
        s[r >> 2][2 * e] += lo;
        s[r >> 2][2 * e + 1] += hi;
        amax[r >> 2] = fmaxf(amax[r >> 2], fmaxf(fabsf(lo), fabsf(hi)));
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    *(float4*)&sums[rg][h][cg * 8] = make_float4(s[h][0], s[h][1], s[h][2], s[h][3]);
    *(float4*)&sums[rg][h][cg * 8 + 4] = make_float4(s[h][4], s[h][5], s[h][6], s[h][7]);
  }
  if (part == 0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      amax[h] = rows_max(row_max(amax[h]));
      if ((t & 63) == 0) s_amax[h][t >> 6] = amax[h];
    }
  }
  __syncthreads();
  const int half = t >> 7, c = t & 127;
  if (part == 2) {
    if (t < 128) {
      float m = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, sums[r][0][t]);
      A.vmax_part[(size_t)blk * D + t] = m;
    }
    return;
  }
  float tot = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) tot += sums[r][half][c];
  const int cnt0 = min(64, max(0, N - row0)), cnt1 = min(64, max(0, N - row0 - 64)), cnt = half ? cnt1 : cnt0;
  if (part == 1) {
    if (cnt > 0) A.kbar[((size_t)bh * A.Tk + 2 * g + half) * D + c] = tot / (float)cnt;
    return;
  }
  if (A.block_q == 64) {
    if (cnt > 0) A.qbar[((size_t)bh * A.Tq + 2 * g + half) * D + c] = tot / (float)cnt;
  } else {
    // both halves belong to query block g: combine the two partial sums
    __syncthreads();
    sums[0][half][c] = tot;
    __syncthreads();
    if (half == 0) A.qbar[((size_t)bh * A.Tq + g) * D + c] = (sums[0][0][c] + sums[0][1][c]) / (float)(cnt0 + cnt1);
  }
  if (t == 0) {
    float m[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) m[h] = fmaxf(fmaxf(s_amax[h][0], s_amax[h][1]), fmaxf(s_amax[h][2], s_amax[h][3]));
    if (A.block_q == 64) {
      if (cnt0 > 0) A.dq[(size_t)bh * A.Tq + 2 * g] = m[0] > 0.f ? m[0] / 127.0f : 1.0f;
      if (cnt1 > 0) A.dq[(size_t)bh * A.Tq + 2 * g + 1] = m[1] > 0.f ? m[1] / 127.0f : 1.0f;
    } else {
      m[0] = m[1] = fmaxf(m[0], m[1]);
      A.dq[(size_t)bh * A.Tq + g] = m[0] > 0.f ? m[0] / 127.0f : 1.0f;
    }
    s_qmax[0] = m[0];
    s_qmax[1] = m[1];
  }
  // ---- INT8 codes of Q at the scale just found (max|Q block| / 127), ties exact: every row's 128 bytes in the
  // order the attention kernel's lanes take them (q8_byte_offset); this thread: 8 adjacent bytes of 8 rows.
  if (A.q8 == nullptr) return;  // (uniform)
  __syncthreads();
  int8_t* dst = A.q8 + ((size_t)blk * 128) * D + q8_byte_offset(cg * 8);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int rl = rg + 16 * r;
    if (row0 + rl >= N) continue;
    const CodeScale cs = code_scale(s_qmax[r >> 2], 127.0f);
    const uint32_t w[4] = {x[r].x, x[r].y, x[r].z, x[r].w};
    uint32_t code[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      code[2 * e] = int8_code_word_exact(bf16_lo(w[e]), cs);
      code[2 * e + 1] = int8_code_word_exact(bf16_hi(w[e]), cs);
    }
    *(uint2*)(dst + (size_t)rl * D) = make_uint2(pack_low_bytes(code[0], code[1], code[2], code[3]), pack_low_bytes(code[4], code[5], code[6], code[7]));
  }
}

__global__ void zero_u32_kernel(uint32_t* p, size_t n) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// What the statistics still need once every block's sums are known; runs as the first workgroups of the scores
// launch (both depend on pool_stats alone, and a launch of its own cost the smallest calls 11 of 61 us).
// Workgroups 0 .. 8 BH - 1, eight per (b,h), each for 16 channels: mu_K[c] = sum_j cnt_j kbar[j][c] / N, max|V[:,c]|,
// delta_V[c] = max|V[:,c]| / 448 (1 if zero).  The INT8 codes of K hang on the last bit of the mean, so its order of
// summation is part of the result (MEAN_RUNS).  A thread carries MEAN_RUNS / 16 of them, which also keeps that many loads in flight.
__device__ __forceinline__ void finalize_block(int blk, const float* __restrict__ kbar, const float* __restrict__ vmax_part,
                                               int groups, int N, int Tk, float* __restrict__ mu_k,
                                               float* __restrict__ amax_v, float* __restrict__ dv) {
  constexpr int PER = MEAN_RUNS / 16;
  __shared__ float sums[MEAN_RUNS][17], maxima[16][17];
  const int bh = blk >> 3, c0 = (blk & 7) * 16, t = threadIdx.x, cl = t & 15, rgrp = t >> 4;
  float s[PER] = {}, m = 0.f;
  const float* col = kbar + (size_t)bh * Tk * D + c0 + cl;
  int j0 = 0;
#pragma unroll 4
  for (; j0 + MEAN_RUNS <= Tk && (j0 + MEAN_RUNS) * BK <= N; j0 += MEAN_RUNS)   // (whole blocks only)
#pragma unroll
    for (int u = 0; u < PER; ++u) s[u] = __builtin_fmaf(col[(size_t)(j0 + rgrp + 16 * u) * D], (float)BK, s[u]);
  for (; j0 < Tk; j0 += MEAN_RUNS)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int j = j0 + rgrp + 16 * u;
      if (j < Tk) s[u] = __builtin_fmaf(col[(size_t)j * D], (float)min(BK, N - j * BK), s[u]);
    }
#pragma unroll 8
  for (int g = rgrp; g < groups; g += 16) m = fmaxf(m, vmax_part[((size_t)bh * groups + g) * D + c0 + cl]);
#pragma unroll
  for (int u = 0; u < PER; ++u) sums[rgrp + 16 * u][cl] = s[u];
  maxima[rgrp][cl] = m;
  __syncthreads();
  if (t < 16) {
    float tot = 0.f;
#pragma unroll
    for (int r = 0; r < MEAN_RUNS; ++r) tot += sums[r][t];
#pragma unroll
    for (int r = 0; r < 16; ++r) m = fmaxf(m, maxima[r][t]);
    const size_t o = (size_t)bh * D + c0 + t;
    mu_k[o] = tot / (float)N;
    amax_v[o] = m;
    dv[o] = m > 0.f ? m / E4M3_MAX : 1.0f;
  }
}
// The output projection (the identity if none is given) in the order in which prep_kv's first product takes it as
// the B operand of v_mfma_f32_32x32x16_bf16: 16-byte chunk [tile of 32 output channels][step of 16 input
// channels][lane] = W[32 tile + lane % 32][16 step + 8 (lane / 32) + 0..7], so that a wavefront fetches an operand as
// one contiguous KiB.  One chunk per thread, WFRAG_BLOCKS workgroups.
constexpr int WFRAG_BLOCKS = D * D / 8 / 256;
__device__ __forceinline__ void wfrag_block(int blk, const bf16_t* __restrict__ proj_w, bf16_t* __restrict__ wfrag) {
  const int idx = blk * 256 + threadIdx.x, lane = idx & 63, row = 32 * (idx >> 9) + (lane & 31), col = 16 * ((idx >> 6) & 7) + 8 * (lane >> 5);
#pragma unroll
  for (int e = 0; e < 8; ++e)
    wfrag[idx * 8 + e] = proj_w ? proj_w[row * D + col + e] : (row == col + e ? (bf16_t)0x3f80 : (bf16_t)0);
}

// scores: s[bh][i][j] = qbar_i . kbar_j / sqrt(d) in fp32 on the matrix pipe
// (v_mfma_f32_32x32x2_f32: fp32 operands and accumulation, the vector-fp32 rate without its issue
// limits).  A wavefront owns a 32-row tile of query blocks, whose means it keeps in registers, and
// sweeps jt_run 32-column tiles of key blocks; the four wavefronts of a workgroup take four
// consecutive row tiles over the SAME columns, so three of their four reads of a key tile hit
// the L1.  The instruction contracts two channels per step, one per lane half; which two is
// free as long as both operands agree: lane half h holds channels 64 h .. 64 h + 63 of its row
// (16 contiguous 16-byte loads) and step t contracts channels t and 64 + t.
typedef float v16f_sc __attribute__((ext_vector_type(16)));
struct ScoresArgs {
  const float *qbar, *kbar;
  float* scores;
  int Tq, Tk, gx, gy, jt_run;     // workgroups per (b,h): gx runs of jt_run column tiles x gy groups of four row tiles
  int fin_blocks, wfrag_blocks;   // leading workgroups that run finalize_block / wfrag_block
  const float* vmax_part;
  int groups, N;
  float *mu_k, *amax_v, *dv;
  const bf16_t* proj_w;
  bf16_t* wfrag;
};
__global__ void __launch_bounds__(256, 2) scores_kernel(const ScoresArgs A) {
  const int first = A.fin_blocks + A.wfrag_blocks;
  if ((int)blockIdx.x < A.fin_blocks) return finalize_block(blockIdx.x, A.kbar, A.vmax_part, A.groups, A.N, A.Tk, A.mu_k, A.amax_v, A.dv);
  if ((int)blockIdx.x < first) return wfrag_block(blockIdx.x - A.fin_blocks, A.proj_w, A.wfrag);
  const int Tq = A.Tq, Tk = A.Tk, blk = blockIdx.x - first, bx = blk % A.gx, by = blk / A.gx % A.gy, bh = blk / (A.gx * A.gy);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l32 = lane & 31, h = lane >> 5;
  const int i0 = (by * 4 + w) * 32;
  if (i0 >= Tq) return;  // (whole wavefront; no barriers in this part of the kernel)
  const int jt0 = bx * A.jt_run, jts = (Tk + 31) / 32;
  float a[64], b[64];
  {
    const float4* src = (const float4*)(A.qbar + ((size_t)bh * Tq + min(i0 + l32, Tq - 1)) * D + 64 * h);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const float4 x = src[u];
      a[4 * u] = x.x; a[4 * u + 1] = x.y; a[4 * u + 2] = x.z; a[4 * u + 3] = x.w;
    }
  }
  auto load_b = [&](int jt) {
    const float4* src = (const float4*)(A.kbar + ((size_t)bh * Tk + min(jt * 32 + l32, Tk - 1)) * D + 64 * h);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const float4 x = src[u];
      b[4 * u] = x.x; b[4 * u + 1] = x.y; b[4 * u + 2] = x.z; b[4 * u + 3] = x.w;
    }
  };
  for (int jt = jt0; jt < min(jt0 + A.jt_run, jts); ++jt) {
    load_b(jt);
    v16f_sc acc = {};
#pragma unroll
    for (int t = 0; t < 64; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[t], acc, 0, 0, 0);
    // accumulator register r of lane (l32, h): row 8 (r / 4) + 4 h + r % 4, column l32
    const int j = jt * 32 + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = i0 + 8 * (r >> 2) + 4 * h + (r & 3);
      if (i < Tq && j < Tk) A.scores[((size_t)bh * Tq + i) * Tk + j] = acc[r] / 11.313708498984761f;
    }
  }
}

template <int KPL>
__global__ void __launch_bounds__(256) select_kernel(const SelectArgs S) {
  const unsigned row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row < (unsigned)S.rows) select_row<KPL>(S, row, ScoresOf{S.scores + (size_t)row * S.Tk});  // (no workgroup barrier: whole wavefronts may leave)
}

// ---------------------------------------------------------------------------
void launch_zero_u32(uint32_t* p, size_t n, hipStream_t stream) {
  zero_u32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(p, n);
}

void launch_pool_stats(const void* q, const void* k, const void* v, const Problem& p, float* qbar,
                       float* kbar, float* dq, float* vmax_part, int8_t* q8, hipStream_t stream) {
  const int groups = (p.N + 127) / 128, per_part = p.BH * groups;
  pool_stats_kernel<<<(v ? 3u : 2u) * (unsigned)per_part, 256, 0, stream>>>(
      PoolArgs{{(const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v}, {p.lq, p.lk, p.lv}, p.N, p.block_q, p.Tq, p.Tk, groups, p.H, per_part,
               qbar, kbar, dq, vmax_part, q8});
}

void launch_scores(const Problem& p, const float* qbar, const float* kbar, float* scores, const FinalizeArgs* fin,
                   hipStream_t stream) {
  ScoresArgs A{};
  A.qbar = qbar; A.kbar = kbar; A.scores = scores;
  A.Tq = p.Tq; A.Tk = p.Tk; A.N = p.N;
  A.groups = (p.N + 127) / 128;
  if (fin) {
    A.vmax_part = fin->vmax_part;
    A.mu_k = fin->mu_k; A.amax_v = fin->amax_v; A.dv = fin->dv;
    A.proj_w = fin->proj_w; A.wfrag = fin->wfrag;
    A.fin_blocks = fin->mu_k ? 8 * p.BH : 0;
    A.wfrag_blocks = fin->wfrag ? WFRAG_BLOCKS : 0;
  }
  int n_scores = 0;
  if (scores) {
    const int jts = (p.Tk + 31) / 32;
    A.gy = (p.Tq + 127) / 128;
    // runs of four column tiles share a wavefront's query means; where those would leave compute units without a
    // workgroup, one tile each (24 slices of 37 x 73 blocks: 24 workgroups, 13.6 us)
    A.jt_run = (long long)((jts + 3) / 4) * A.gy * p.BH >= 512 ? 4 : 1;
    A.gx = (jts + A.jt_run - 1) / A.jt_run;
    n_scores = A.gx * A.gy * p.BH;
  }
  const int grid = A.fin_blocks + A.wfrag_blocks + n_scores;
  if (grid > 0) scores_kernel<<<(unsigned)grid, 256, 0, stream>>>(A);
}

void launch_select(const Problem& p, const float* scores, int8_t* mask, int32_t* crit, int32_t* marg,
                   uint32_t* mbits, hipStream_t stream) {
  const int rows = p.BH * p.Tq, need = (p.Tk + 63) / 64;
  const SelectArgs S{scores, rows, p.Tq, p.Tk, p.n_c, p.n_m, mask, crit, marg, mbits};
#define SLA_SELECT(K) select_kernel<K><<<(unsigned)((rows + 3) / 4), 256, 0, stream>>>(S)
  // registers per lane: the smallest instantiation that holds the row
  if (need <= 2) SLA_SELECT(2);
  else if (need <= 4) SLA_SELECT(4);
  else if (need <= 8) SLA_SELECT(8);
  else if (need <= 12) SLA_SELECT(12);
  else if (need <= 16) SLA_SELECT(16);
  else if (need <= 20) SLA_SELECT(20);
  else if (need <= 24) SLA_SELECT(24);
  else if (need <= 32) SLA_SELECT(32);
  else if (need <= 48) SLA_SELECT(48);
  else if (need <= 64) SLA_SELECT(64);
  else if (need <= 96) SLA_SELECT(96);
  else SLA_SELECT(128);
#undef SLA_SELECT
}

}  // namespace sla
