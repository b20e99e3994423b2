// prep_kv: per key block, the operands of both branches.
//
//  * Low-bit sparse branch (Section 1.1 names the scheme; the granularity is this
//    library's reading, see sla.h): K~ = K - mean_K, INT8 codes with one scale per key
//    block; V / delta_V[c] as FP8 E4M3 codes.  Both are written in MFMA fragment order
//    (common.h) so the attention kernel stages them with straight 16-byte copies.
//  * Linear branch: with phi the per-token feature map on the ORIGINAL K,
//        hz[o][c] = sum_rows (V W^T)[row][o] * phi(K)[row][c]   (o < 128)
//        hz[128][c] = sum_rows phi(K)[row][c]
//    i.e. the block summary h_j with the output projection already folded in
//    (transposed, c contiguous) and z_j as row 128.  Two bf16 MFMA products with fp32
//    accumulation; the first product's accumulators are fed to the second as its A
//    operand directly from registers (the contraction order of the second product is
//    permuted to match, for both operands).
//
// One workgroup (4 wavefronts) per (b,h,j): reads 32 KiB, writes 16 KiB of codes and 33 KiB of summaries.  With the staged codes
// and phi(K) spread over the banks (a row's codes met in four: of 344 M LDS cycles at 40 x 75600 tokens 234 M were conflicts, now 32
// of 100 M) and reductions on the vector ALU instead of through LDS the launch, selection included, takes 699 us there (before: 816),
// 5.5 TB/s, what a large copy gets; 102 at 12 x 32760 (122), 29.7 at 24 x 4617 (41.4); there, with 6 to 8 wavefronts' worth of
// instructions per SIMD, by issuing them.
#include "classify.h"
#include "delta.h"

namespace sla {

struct MidArgs {
  SelectArgs S;
  DeltaArgs X;
  PrepArgs P;
  int select_blocks, delta_blocks;   // leading workgroups of the selection, then those of delta
};

constexpr int STAGE_STRIDE = 2 * D + 16;  // bytes per staged hz row (padded against bank conflicts)

// Where bytes of a K or V record (at offset o) and 16-byte chunk q of phi(K)^T are staged in LDS: the chunks are permuted
// within groups of 8 and 16, or the lanes that write a row's codes, or the same row of 16 channels, would meet in four banks
// of 64 (16 lanes in each).
__device__ __forceinline__ int staged_code(int o) {
  const int p = o >> 4;
  return o ^ (((((p >> 4) ^ (p >> 6)) & 1) | ((p >> 5) & 1) << 1 | ((p >> 7) & 1) << 2) << 4);
}
__device__ __forceinline__ int staged_phi(int q) { return (q ^ ((q >> 4) & 15)) << 4; }

// The statistics of slice bh joined over its (at most MEAN_RUNS) key blocks: stat[c] = mean of K, stat[128 + c] = max|V|.  The
// sums are finalize_block's, in its order.
__device__ __forceinline__ void slice_stats(const PrepArgs& P, int bh, bool publish, float* stat) {
  const int t = threadIdx.x, c = t & 127, N = P.N, Tk = P.Tk;
  if (t < 128) {
    const float* col = P.kbar + (size_t)bh * Tk * D + c;
    float tot = 0.f;
#pragma unroll 16
    for (int r = 0; r < Tk; ++r) tot += __builtin_fmaf(col[(size_t)r * D], (float)min(BK, N - r * BK), 0.f);
    stat[c] = tot / (float)N;
    if (publish) P.mu_out[(size_t)bh * D + c] = stat[c];
  } else {
    float m = 0.f;
#pragma unroll 8
    for (int g = 0; g < P.groups; ++g) m = fmaxf(m, P.vmax_part[((size_t)bh * P.groups + g) * D + c]);
    stat[D + c] = m;
    if (publish) {
      P.amax_out[(size_t)bh * D + c] = m;
      P.dv_out[(size_t)bh * D + c] = m > 0.f ? m / E4M3_MAX : 1.0f;
    }
  }
}
// Row `row` of W (the identity if no projection is given) as product 1's operands, columns 16 ks + col .. + 7, straight
// from the caller's matrix.  (One test for all of them: behind a test each they waited for memory one by one.)
__device__ __forceinline__ void w_operands(const PrepArgs& P, int row, int col, v8bf (&out)[8]) {
  if (P.w_aligned) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) out[ks] = *(const v8bf*)(P.proj_w + row * D + 16 * ks + col);
  } else {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      union { bf16_t e[8]; v8bf v; } x;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = 16 * ks + col + e;
        x.e[e] = P.proj_w ? P.proj_w[row * D + c] : (row == c ? (bf16_t)0x3f80 : (bf16_t)0);
      }
      out[ks] = x.v;
    }
  }
}
// The four query blocks 4 blk .. 4 blk + 3 of a slice, one per wavefront: the scores against all (at most 64) key blocks, one per
// lane, then the selection, without LDS.  scores_kernel's matrix product adds up channels t and 64 + t step by step, and
// an fp32 product of the matrix pipe is a chain of fused operations: so are these, in the same order, bit for bit the same
// (on 32 rows of which 28 were copies the product alone took 4096 cycles: training step of 4 x 2187 tokens 118.5 -> 114.0 us).
__device__ __forceinline__ void classify_rows(const SelectArgs& S, const float* __restrict__ qbar, const float* __restrict__ kbar, int blk) {
  const int Tq = S.Tq, Tk = S.Tk, per = (Tq + 3) / 4, bh = blk / per;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = 4 * (blk - bh * per) + w;
  if (i >= Tq) return;               // (whole wavefront; no barriers here)
  const unsigned row = (unsigned)(bh * Tq + i);
  // (uniform, and written by an earlier launch: through the scalar unit)
  const __attribute__((address_space(4))) float* qrow = (const __attribute__((address_space(4))) float*)(uintptr_t)(qbar + (size_t)row * D);
  const float4* krow = (const float4*)(kbar + ((size_t)bh * Tk + min(lane, Tk - 1)) * D);
  float sum = 0.f;
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    float4 lo[8], hi[8];             // channels 32 part .. + 31 and 64 on
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      lo[u] = krow[8 * part + u];
      hi[u] = krow[16 + 8 * part + u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float b0[4] = {lo[u].x, lo[u].y, lo[u].z, lo[u].w}, b1[4] = {hi[u].x, hi[u].y, hi[u].z, hi[u].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 32 * part + 4 * u + e;
        sum = __builtin_fmaf(qrow[c], b0[e], sum);
        sum = __builtin_fmaf(qrow[64 + c], b1[e], sum);
      }
    }
  }
  const float score = sum / 11.313708498984761f;
  select_row<1>(S, row, [&](int) { return score; });
}

// STATS (calls of few key blocks): nobody has joined the statistics over the slice yet or laid out W; every workgroup does
// that for itself (mean of K and max|V| of at most 64 key blocks, W's operands from where they are).
template <int PHI, bool STATS>
__device__ __forceinline__ void prep_block(const PrepArgs& P, int blk) {
  const bf16_t *k = P.k, *v = P.v, *wfrag = P.wfrag;
  const int N = P.N, Tk = P.Tk, H = P.H, want_quant = P.want_quant, want_linear = P.want_linear;
  const Layout &lk = P.lk, &lv = P.lv;
  int8_t* k8 = P.k8;
  uint8_t* v8 = P.v8;
  float* dk = P.dk;
  bf16_t* hz = P.hz;
  __shared__ __attribute__((aligned(16))) unsigned char smem[128 * STAGE_STRIDE + 4 * D * 4];
  __shared__ float wave_amax[4];
  unsigned char* kq = smem;                       // [8192]  K codes, fragment order
  unsigned char* vq = smem + KV_FRAG_BYTES;       // [8192]  V codes, fragment order
  unsigned char* vbf = smem;                      // [64][STAGE_STRIDE] V rows as bf16 (aliases kq / vq, after their last read)
  unsigned char* phit = smem + BK * STAGE_STRIDE; // [16384] phi(K)^T bf16, B-operand order
  unsigned char* stage = smem;                    // [128][STAGE_STRIDE] aliases everything above
  float* zred = (float*)(smem + 128 * STAGE_STRIDE);  // [4][128] per-wavefront column sums of phi(K); before that STATS' mean and maxima

  const int bh = blk / Tk, j = blk % Tk;
  const int t = threadIdx.x, cg = t & 15, m = t >> 4, lane = t & 63, w = t >> 6;
  const int valid = min(BK, N - j * BK);
  const int b_ = bh / H, h_ = bh - b_ * H;
  const bf16_t* kblk = k + b_ * lk.sb + h_ * lk.sh + (long long)j * BK * lk.sn;
  const bf16_t* vblk = v + b_ * lv.sb + h_ * lv.sh + (long long)j * BK * lv.sn;

  float kf[4][8];
  uint4 kraw[4], vraw[4];  // V stays packed: it is quantised from these words and staged for product 1 as they are
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * m + r;
    kraw[r] = vraw[r] = make_uint4(0, 0, 0, 0);
    if (row < valid) {
      kraw[r] = *(const uint4*)(kblk + row * lk.sn + cg * 8);
      vraw[r] = *(const uint4*)(vblk + row * lv.sn + cg * 8);
    }
  }
  if constexpr (STATS) {             // (under way together with the rows)
    if (want_quant) slice_stats(P, bh, j == 0, zred);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t wk[4] = {kraw[r].x, kraw[r].y, kraw[r].z, kraw[r].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      kf[r][2 * e] = bf16_lo(wk[e]);
      kf[r][2 * e + 1] = bf16_hi(wk[e]);
    }
  }

  if (want_quant) {
    const float *mu_k = P.mu_k + (size_t)bh * D, *amax_v = P.amax_v + (size_t)bh * D;
    if constexpr (STATS) {
      mu_k = zred;
      amax_v = zred + D;
      __syncthreads();
    }
    float mu[8];
    CodeScale vcs[8];  // per channel: max|V| (its scale is this / 448), its reciprocal, 448
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mu[e] = mu_k[cg * 8 + e];
      vcs[e] = code_scale(amax_v[cg * 8 + e], E4M3_MAX);
    }
    float kt[4][8], amax = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        kt[r][e] = (4 * m + r < valid) ? kf[r][e] - mu[e] : 0.f;
        amax = fmaxf(amax, fabsf(kt[r][e]));
      }
    amax = rows_max(row_max(amax));
    if (lane == 0) wave_amax[w] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(wave_amax[0], wave_amax[1]), fmaxf(wave_amax[2], wave_amax[3]));
    const float delta = amax > 0.f ? amax / 127.0f : 1.0f;
    // K codes by multiplication with the reciprocal: differs from a true division only at
    // rounding ties, where one INT8 step moves a score by delta_Q delta_K (the FP8 V codes, whose
    // steps are coarse, keep the true division).  Adding 1.5 * 2^23 inside the fma rounds the
    // product to the nearest integer (ties to even) and leaves its two's-complement low byte in
    // the low byte of the float; |k~ / delta| <= 127 by construction, so no clamp is needed.
    const float inv_delta = 1.0f / delta;
    if (t == 0) dk[(size_t)bh * Tk + j] = delta;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      uint32_t b[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = __float_as_uint(__builtin_fmaf(kt[r][e], inv_delta, 12582912.0f));
      const uint32_t lo = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u),
                                                __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), 0x05040100u);
      const uint32_t hi = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[7], b[6], 0x0c0c0400u),
                                                __builtin_amdgcn_perm(b[5], b[4], 0x0c0c0400u), 0x05040100u);
      *(uint2*)(kq + staged_code(kfrag_offset(4 * m + r, cg * 8))) = make_uint2(lo, hi);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // v / delta_V = 448 v / max|V|: the product 448 v is exact for a 16-bit v, and reciprocal + one
        // correction step (the fma forms the residual exactly) gives the correctly rounded quotient, so a
        // value exactly half way between two FP8 values reaches the conversion as the tie it is -- at a
        // third of the cost of the general division sequence
        const uint32_t word = (e >> 1) == 0 ? vraw[r].x : (e >> 1) == 1 ? vraw[r].y : (e >> 1) == 2 ? vraw[r].z : vraw[r].w;
        const float qv = exact_quotient((e & 1) ? bf16_hi(word) : bf16_lo(word), vcs[e]);
        x[r] = clamp_e4m3(qv);
      }
      int code = cvt_pk_e4m3(x[0], x[1], 0, false);
      code = cvt_pk_e4m3(x[2], x[3], code, true);
      *(int*)(vq + staged_code(vfrag_offset(4 * m, cg * 8 + e))) = code;
    }
    __syncthreads();
    const size_t rec = ((size_t)bh * Tk + j) * KV_FRAG_BYTES;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int o = (u * 256 + t) * 16;
      *(uint4*)(k8 + rec + o) = *(const uint4*)(kq + staged_code(o));
      *(uint4*)(v8 + rec + o) = *(const uint4*)(vq + staged_code(o));
    }
  }
  if (!want_linear) return;

  // ---- phi(K): rows live across the 16 lanes that share m
  float ph[4][8];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const bool ok = 4 * m + r < valid;
    if (PHI == 0) {
      float mx = kf[r][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) mx = fmaxf(mx, kf[r][e]);
      mx = row_max(mx);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ph[r][e] = __builtin_amdgcn_exp2f((kf[r][e] - mx) * LOG2E);
        s += ph[r][e];
      }
      s = row_sum(s);
      const float inv = ok ? 1.0f / s : 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) ph[r][e] *= inv;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = kf[r][e];
        float y;
        if (PHI == 1) y = x > 0.f ? x + 1.0f : __builtin_amdgcn_exp2f(x * LOG2E);
        else y = fmaxf(x, 0.f);
        ph[r][e] = ok ? y : 0.f;
      }
    }
  }
  __syncthreads();  // kq / vq reads are done; phit may now be written
  {
    const int tt = m >> 3, g = (m & 7) >> 1, hf = m & 1, s2 = tt * 2 + (g >> 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = cg * 8 + e;
      const uint2 pk = make_uint2(pack_bf16x2(ph[0][e], ph[1][e]), pack_bf16x2(ph[2][e], ph[3][e]));
      *(uint2*)(phit + staged_phi((s2 * 128 + c) * 2 + hf) + (g & 1) * 8) = pk;
      float zs = ph[0][e] + ph[1][e] + ph[2][e] + ph[3][e];  // 4 rows of this thread, then the 4 row groups of the wavefront
      zs = rows_sum(zs);
      if (lane < 16) zred[w * D + c] = zs;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) *(uint4*)(vbf + (4 * m + r) * STAGE_STRIDE + cg * 16) = vraw[r];
  }
  const int hfl = lane >> 5, l32 = lane & 31;
  v8bf wop[8];   // this wavefront's 32 rows of W
  if constexpr (STATS) w_operands(P, 32 * w + l32, 8 * hfl, wop);
  else {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) wop[ks] = *(const v8bf*)(wfrag + ((w * 8 + ks) * 64 + lane) * 8);
  }
  __syncthreads();  // phit, zred and the V rows are complete

  // ---- product 1: VW[row][o] for o in this wavefront's tile of 32 output channels
  v16f d1[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    d1[rt] = v16f{};
    const int row = 32 * rt + l32;  // rows past the end of a ragged block were staged as zeros
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const v8bf a = *(const v8bf*)(vbf + row * STAGE_STRIDE + 32 * ks + 16 * hfl);
      d1[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, wop[ks], d1[rt], 0, 0, 0);
    }
  }

  // ---- product 2, transposed: hz^T[c][o] = sum over rows of phi[row][c] VW[row][o], so that a lane
  // ends up with four consecutive c of one o in consecutive registers (8-byte staging writes)
  v16f d2[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) d2[ct] = v16f{};
#pragma unroll
  for (int s2 = 0; s2 < 4; ++s2) {
    v8bf a;
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = (__bf16)d1[s2 >> 1][8 * (s2 & 1) + e];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const v8bf b = *(const v8bf*)(phit + staged_phi((s2 * 128 + 32 * ct + l32) * 2 + hfl));
      d2[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, d2[ct], 0, 0, 0);
    }
  }
  float zsum = 0.f;
  if (t < D) {
#pragma unroll
    for (int r = 0; r < 4; ++r) zsum += zred[r * D + t];
  }
  __syncthreads();  // every wavefront is done reading phit: the staging area may overwrite it
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v16f& x = d2[ct];
      *(uint2*)(stage + (32 * w + l32) * STAGE_STRIDE + (32 * ct + 8 * g + 4 * hfl) * 2) =
          make_uint2(pack_bf16x2(x[4 * g], x[4 * g + 1]), pack_bf16x2(x[4 * g + 2], x[4 * g + 3]));
    }
  __syncthreads();
  bf16_t* dst = hz + ((size_t)bh * Tk + j) * HZ_ELEMS;
  // h'^T leaves in the order in which the attention kernel's epilogue takes it as the A operand of
  // v_mfma_f32_32x32x16_bf16 (hz_frag_chunk in common.h); the accumulation over marginal blocks in
  // between is element-wise and does not care.  16-byte chunk d of the destination = row o,
  // channels 8 cq .. 8 cq + 7 of the staged tile.
  for (int d = t; d < 128 * 16; d += 256) {
    const int ot = d >> 9, ks = (d >> 6) & 7, ln = d & 63;
    const int o = 32 * ot + (ln & 31), cq = 4 * (ks >> 1) + 2 * (ln >> 5) + (ks & 1);
    *(uint4*)(dst + d * 8) = *(const uint4*)(stage + o * STAGE_STRIDE + cq * 16);
  }
  if (t < D) dst[D * D + t] = f32_to_bf16(zsum);
}

// One launch for everything that only waits for the statistics pass (and, without STATS, for the scores): the selection
// of the critical and marginal blocks, delta = dO . O^s of a backward pass with saved state, and the workgroups of
// prep_block.  They need nothing of one another, and the selection, which is all compares and latency, runs under
// prep_block's traffic (its workgroups first; spread among prep_block's they were 2 to 5 % slower).
// STATS: the scores themselves are formed here as well, four query blocks per workgroup.
template <int PHI, int KPL, bool STATS>
__global__ void __launch_bounds__(256, 4) select_prep_kernel(const MidArgs A) {
  int blk = blockIdx.x;
  if (blk < A.select_blocks) {
    if constexpr (STATS) {
      static_assert(KPL == 1, "a key block per lane");
      classify_rows(A.S, A.P.qbar, A.P.kbar, blk);
    } else {
      const unsigned row = (unsigned)blk * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      if (row < (unsigned)A.S.rows) select_row<KPL>(A.S, row, ScoresOf{A.S.scores + (size_t)row * A.S.Tk});
    }
    return;
  }
  blk -= A.select_blocks;
  if (blk < A.delta_blocks) return delta_block(A.X, blk);
  prep_block<PHI, STATS>(A.P, blk - A.delta_blocks);
}

// Plain-layout copies of the codes (tests only).
__global__ void unfragment_kv_kernel(const int8_t* __restrict__ k8, const uint8_t* __restrict__ v8,
                                     int N, int Tk, int8_t* __restrict__ k_codes,
                                     uint8_t* __restrict__ v_codes) {
  const int bh = blockIdx.x / Tk, j = blockIdx.x % Tk;
  const size_t rec = ((size_t)bh * Tk + j) * KV_FRAG_BYTES;
  for (int e = threadIdx.x; e < BK * D; e += blockDim.x) {
    const int key = e / D, ch = e % D;
    const int row = j * BK + key;
    if (row >= N) continue;
    const size_t o = ((size_t)bh * N + row) * D + ch;
    if (k_codes) k_codes[o] = k8[rec + kfrag_offset(key, ch)];
    if (v_codes) v_codes[o] = v8[rec + vfrag_offset(key, ch)];
  }
}

__global__ void unpack_q8_kernel(const int8_t* __restrict__ q8, int N, int q8_rows, size_t total, int8_t* __restrict__ q_codes) {
  const size_t x = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (x >= total) return;
  const int ch = (int)(x % D);
  const size_t row = (x / D) % N, bh = x / ((size_t)D * N);
  q_codes[x] = q8[(bh * q8_rows + row) * D + q8_byte_offset(ch)];
}

// SLA_QUANT_QK_INT8: the INT8 codes of Q and of the smoothed K as bf16 numbers (integers up to 127
// are exact in bf16), [BH, N, D] contiguous, for the 16-bit attention kernel: its products of such
// operands are the integer products, exactly (|sum| < 2^24 in the fp32 accumulator).
// One workgroup per key block; the same for the query rows it covers.
__global__ void __launch_bounds__(256) code_tensors_kernel(const int8_t* __restrict__ q8, const int8_t* __restrict__ k8,
                                                           int N, int Tk, int q8_rows, bf16_t* __restrict__ qc,
                                                           bf16_t* __restrict__ kc) {
  const int bh = blockIdx.x / Tk, j = blockIdx.x % Tk;
  const size_t rec = ((size_t)bh * Tk + j) * KV_FRAG_BYTES;
  for (int e = threadIdx.x; e < BK * D; e += 256) {
    const int key = e / D, ch = e % D, row = j * BK + key;
    if (row >= N) continue;
    const size_t o = ((size_t)bh * N + row) * D + ch;
    kc[o] = f32_to_bf16((float)k8[rec + kfrag_offset(key, ch)]);
    qc[o] = f32_to_bf16((float)q8[((size_t)bh * q8_rows + row) * D + q8_byte_offset(ch)]);  // the low-bit kernel's own codes
  }
}

__global__ void e4m3_encode_kernel(const float* __restrict__ in, uint8_t* __restrict__ out, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = (uint8_t)(cvt_pk_e4m3(clamp_e4m3(in[i]), 0.f, 0, false) & 0xff);
}

PrepArgs prep_args(const void* k, const void* v, const Problem& p, const float* mu_k, const float* amax_v, const bf16_t* wfrag,
                   bool want_quant, bool want_linear, int8_t* k8, uint8_t* v8, float* dk, bf16_t* hz) {
  PrepArgs P{};
  P.k = (const bf16_t*)k; P.v = (const bf16_t*)v;
  P.N = p.N; P.Tk = p.Tk; P.H = p.H; P.lk = p.lk; P.lv = p.lv;
  P.mu_k = mu_k; P.amax_v = amax_v; P.wfrag = wfrag;
  P.want_quant = want_quant; P.want_linear = want_linear;
  P.k8 = k8; P.v8 = v8; P.dk = dk; P.hz = hz;
  return P;
}

void launch_prep_kv(const PrepArgs& P, const Problem& p, int phi_kind, hipStream_t stream) {
  MidArgs A{};
  A.P = P;
  const unsigned grid = (unsigned)(p.BH * p.Tk);
  if (phi_kind == 0) select_prep_kernel<0, 2, false><<<grid, 256, 0, stream>>>(A);
  else if (phi_kind == 1) select_prep_kernel<1, 2, false><<<grid, 256, 0, stream>>>(A);
  else select_prep_kernel<2, 2, false><<<grid, 256, 0, stream>>>(A);
}

// One launch for scores, selection and operands where a slice has at most 64 key blocks (2 slices of 128 blocks, us for the whole
// forward call, two launches / one: 55.6 / 57.0) and the workgroups of the key blocks, which all join their slice's statistics for
// themselves, stand on the chip at once, four on a compute unit: later ones repeat it behind those.  Slices x key blocks: 16 x 64 in
// blocks of 64 69.7 / 68.3, of 128 67.6 / 67.0, 32 x 32 70.5 / 68.1 and 64.0 / 61.1, 64 x 16 66.3 / 64.0 and 60.1 / 56.3, 2 x 64 39.1 /
// 34.4; but 20 x 64 85.3 / 88.0 and 81.6 / 81.9, 32 x 40 85.4 / 88.1 and 80.7 / 82.7, 64 x 24 96.3 / 100.1 and 93.8 / 94.9, 40 x 64 164.2 /
// 169.3 and 150.9 / 154.0, 64 x 56 230.5 / 246.4 and 218.3 / 230.5.  Up to 16 key blocks there is little to join, and the line lies where
// the workgroups of four query blocks are few: 96 x 16 (384 of them in blocks of 64) 95.2 / 93.5 and 86.4 / 82.9, 128 x 16 (512 and 256)
// 1.00 and 0.97 of the time; 150 x 10 (450) 1.02, 200 x 14 (800) 1.05.  (Training steps, which do not quantise, take 0.98 to 1.00 of
// the time on either side.)
bool stats_in_prep(const Problem& p) {
  return p.Tk <= 64 && ((long long)p.BH * p.Tk <= 4 * compute_units() || (p.Tk <= 16 && (long long)p.BH * ((p.Tq + 3) / 4) <= 384));
}

// Long rows are selected in a launch of their own: 40 slices of 591 x 1182 blocks take 163 us there and 1003 us with
// prep_block's, in one launch 1020 (prep_block's shared memory leaves the selection half of the wavefronts it hides
// its latency with).  Up to 512 blocks one launch is never slower (everything before the attention kernel in us, two / one: 12
// slices of 256 x 512 288 / 270, 40 of 256 x 512 847 / 835, 40 of 512 x 512 1046 / 1045); instances for longer rows would still
// help few slices (2 of 350 x 700 110 / 89, 12 of 450 x 900 565 / 550) and not many (40 of 700 x 700 1585 / 1593).
bool select_in_prep(const Problem& p) { return p.Tk <= 8 * 64; }

void launch_select_prep(const SelectArgs& S, const PrepArgs& P, const DeltaArgs* delta, const Problem& p, int phi_kind, hipStream_t stream) {
  MidArgs A{};
  A.S = S; A.P = P;
  const bool stats = stats_in_prep(p);
  const int need = (p.Tk + 63) / 64;
  if (delta) {
    A.X = *delta;
    A.delta_blocks = delta_blocks(p);
  }
  if (select_in_prep(p)) A.select_blocks = stats ? p.BH * ((p.Tq + 3) / 4) : (S.rows + 3) / 4;
  const unsigned grid = (unsigned)(A.select_blocks + A.delta_blocks + p.BH * p.Tk);
#define SLA_MID(PHI) { if (stats) select_prep_kernel<PHI, 1, true><<<grid, 256, 0, stream>>>(A); \
                       else if (need <= 2) select_prep_kernel<PHI, 2, false><<<grid, 256, 0, stream>>>(A); \
                       else select_prep_kernel<PHI, 8, false><<<grid, 256, 0, stream>>>(A); }
  if (phi_kind == 0) SLA_MID(0) else if (phi_kind == 1) SLA_MID(1) else SLA_MID(2)
#undef SLA_MID
}

void launch_unfragment_kv(const Problem& p, const int8_t* k8, const uint8_t* v8, int8_t* k_codes,
                          uint8_t* v_codes, hipStream_t stream) {
  unfragment_kv_kernel<<<p.BH * p.Tk, 256, 0, stream>>>(k8, v8, p.N, p.Tk, k_codes, v_codes);
}

void launch_unpack_q8(const Problem& p, const int8_t* q8, int8_t* q_codes, hipStream_t stream) {
  const size_t total = (size_t)p.BH * p.N * D;
  unpack_q8_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(q8, p.N, (p.N + 127) / 128 * 128, total, q_codes);
}

void launch_code_tensors(const Problem& p, const int8_t* q8, const int8_t* k8, bf16_t* qc, bf16_t* kc, hipStream_t stream) {
  code_tensors_kernel<<<p.BH * p.Tk, 256, 0, stream>>>(q8, k8, p.N, p.Tk, (p.N + 127) / 128 * 128, qc, kc);
}

void launch_e4m3_encode(const float* in, uint8_t* out, size_t n, hipStream_t stream) {
  if (n == 0) return;
  e4m3_encode_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(in, out, n);
}

}  // namespace sla
