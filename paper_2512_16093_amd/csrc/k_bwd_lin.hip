// Backward pass of SLA, linear branch and projection (Section 1.2; the forward pass it differentiates:
//     a = phi(Q[n]),  num = a H_i,  den = a . Z_i,  O^l[n] = num / den,   O += O^l W^T + b,
//     H_i = sum_{j marginal for i} phi(K_j)^T V_j,   Z_i = sum_{j marginal for i} sum_t phi(K_j[t]),
// phi = softmax over the channels).
//
//   bwd_lin_q_kernel   per query block i (a workgroup walks over several and keeps dW, db in
//                      registers): dO^l = dO W, dnum = dO^l / den, dden = -(dO^l . O^l) / den,
//                      d phi(Q) = dnum H_i^T + dden Z_i -> dQ (softmax backward), and the block's
//                      dH_i = a^T dnum, dZ_i = a^T dden, written in the summaries' storage order so
//                      that the forward's accumulation kernel can sum them over the transposed mask.
//   (the key side -- per key block j, with G_j = sum_{i : j marginal for i} dH_i and the dZ sum:
//   d phi(K) = V G_j^T + dZ -> dK, dV = phi(K) G_j -- is the prologue of the dK/dV kernel, k_bwd.hip)
//
// As in the sparse-branch kernels a wavefront owns 32 tokens, one per lane pair, and every product
// is formed with the tokens as accumulator columns, so per-token reductions stay in a lane pair.
#include <algorithm>

#include "common.h"

namespace sla {

namespace {

// Where entry [o][c .. c+3] (c a multiple of 4) of a 128 x 128 summary sits in the storage order of
// hz / HZ (hz_frag_chunk): element offset of the 4-element run.
__device__ __forceinline__ int hz_run_offset(int o, int c) {
  const int G = c >> 3, ks = 2 * (G >> 2) + (G & 1), lanep = (o & 31) + 32 * ((G >> 1) & 1);
  return hz_frag_chunk(o >> 5, ks, lanep) * 8 + (c & 7);
}

// Softmax over the 128 channels of this lane pair's token; x holds the lane's 64 channels.
// Returns the row maximum and 1 / sum(exp) through the references; x becomes exp(x - max).
__device__ __forceinline__ void softmax_stats(float (&x)[64], float& mx, float& rsum) {
  mx = x[0];
#pragma unroll
  for (int e = 1; e < 64; ++e) mx = fmaxf(mx, x[e]);
  mx = fmaxf(mx, partner_f32(mx));
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 64; ++e) {
    x[e] = __builtin_amdgcn_exp2f((x[e] - mx) * LOG2E);
    s += x[e];
  }
  s += partner_f32(s);
  rsum = 1.0f / s;
}

}  // namespace

// Workgroup barrier that publishes LDS writes and retires LDS reads but leaves global loads and stores in flight
// (__syncthreads() drains them: five times per query block it then waited for stores nobody in the workgroup reads).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Column sums over the tokens of a staged [BQ][128] tile, weighted: thread (channel group t % 16, ROWS tokens from
// ROWS (t / 16)) adds its share to s[0..7]; tile_sums_finish adds the shares up (wavefront by wavefront into red).
template <int ROWS, class F>
__device__ __forceinline__ void tile_sums(const unsigned char* tile, int t, float (&s)[8], F weight) {
  const int cg = t & 15, n0 = ROWS * (t >> 4);
#pragma unroll
  for (int m = 0; m < ROWS; ++m) {
    float x[8];
    unpack8(*(const uint4*)(tile + (n0 + m) * TP + cg * 16), x);
    const float wm = weight(n0 + m);
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = __builtin_fmaf(x[e], wm, s[e]);
  }
}
__device__ __forceinline__ void tile_sums_finish(float (&s)[8], float* red, int lane, int w) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    s[e] += __shfl_xor(s[e], 16);
    s[e] += __shfl_xor(s[e], 32);
  }
  if (lane < 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[w * 128 + 8 * lane + e] = s[e];
  }
}

// Per query block (BQ tokens): 33 KB of summaries, 2 x 32 KB of Q and dO in, 64 KB of dQ's share (fp32) and 33 KB of
// dH out (BQ = 128) against 160 matrix products per wavefront: bound by memory if nothing else is waited for.  One
// workgroup per compute unit walks over a contiguous run of (head, query block) items; the next item's summaries, Q
// and dO are on their way into registers while the present one is computed, stores are never waited for, and every
// operand that contracts over a tile's rows comes from the row-major tile by the transposing read.  (Before: loads,
// stores and barriers of an item one after the other, transposed copies made by 2-byte writes:
// 40 heads x 75600 tokens 2.82 -> 1.49 ms, 12 x 32760 385 -> 219 us, 4 x 2187 (blocks of 64) 41 -> 29 us.)
//
// TT wavefronts own 32 tokens each, and CS of them share a token, each with 4 / CS of the output tiles.  Query blocks of
// 128 take four with all tiles.  Of 64, two wavefronts left half of the SIMDs idle, with twice the dW and dH tiles each
// (spilled registers, summaries not requested ahead): there four, a pair per token; what it does not share
// (softmax, loads of its rows) is done twice, the two token-wise sums and dnum meet in LDS.  The backward pass of 12 x 32760
// in blocks of 64 4290 -> 4040 us, of 4 x 2187 128 -> 119 us.  (Pairs for blocks of 128 as well, two wavefronts per SIMD: 50
// registers spilled, 3515 -> 3615 us.)
template <int TT, int CS, int PHI>
__global__ void __launch_bounds__(TT * CS * 64, 1)
    bwd_lin_q_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ dout, const bf16_t* __restrict__ HZ,
                     const bf16_t* __restrict__ proj_w, float* __restrict__ dq_lin, bf16_t* __restrict__ dHZ,
                     float* __restrict__ dW_part, float* __restrict__ db_part, int N, int Tq, int total, int H, Layout lq, Layout ld) {
  constexpr int BQ = 32 * TT, NW = CS * TT, NT = 64 * NW, PER = 2048 / NT, OT = 4 / CS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* const Wl = smem;              // W[r][c] (the identity when there is no projection)
  unsigned char* const Hl = Wl + 128 * TP;     // H[o][c]            -> dO[n][r]
  unsigned char* const Al = Hl + 128 * TP;     // a[n][c]            -> O^l[n][c]
  unsigned char* const Dl = Al + BQ * TP;      // dnum[n][o]
  float* const zv = (float*)(Dl + BQ * TP);    // Z[c]
  float* const dden_s = zv + 128;              // dden[n]
  float* const red = dden_s + 128;             // [NW][128]
  float* const half_dden = red + NW * 128;     // [CS][BQ] each (CS > 1): a token's sums over either half of the channels
  float* const half_sdot = half_dden + CS * BQ;
  const int t = threadIdx.x, lane = t & 63, w = CS == 1 ? t >> 6 : __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  // (w in a scalar register costs the instance without shared tokens 0.5 % of its call, 12 x 32760)
  const int ch = CS == 1 ? 0 : w / TT;         // this wavefront's share of the channels: output tiles from OT ch on
  const int nl = 32 * (w - ch * TT) + l32;     // this lane pair's token within the query block
  const int tr_off = tr_lane_offset(lane);
  const int first = (int)((long long)total * blockIdx.x / gridDim.x), end = (int)((long long)total * (blockIdx.x + 1) / gridDim.x);

  if (proj_w && ((uintptr_t)proj_w & 15) == 0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = u * NT + t;
      *(uint4*)(Wl + (x >> 4) * TP + (x & 15) * 16) = *(const uint4*)(proj_w + x * 8);
    }
  } else {
    for (int x = t; x < D * D; x += NT)
      *(bf16_t*)(Wl + (x >> 7) * TP + (x & 127) * 2) = proj_w ? proj_w[x] : (bf16_t)((x >> 7) == (x & 127) ? 0x3F80 : 0);
  }

  static_assert(NW == 4, "of dH and dW a wavefront forms four tiles: row (dW) or column (dH) w of them");
  constexpr int TILES = 4;
  v16f dwacc[TILES];
#pragma unroll
  for (int x = 0; x < TILES; ++x) dwacc[x] = v16f{};
  // (names the sums' place: left alone the allocator moved them between ordinary registers and scratch memory, whose
  // reloads waited for every load and store in flight)
  auto hold_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < TILES; ++x) asm volatile("" : "+a"(dwacc[x]));
  };
  float dbacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // The next item's summaries and rows (rows beyond N come as row N - 1 and are given no weight).
  uint4 hzp[PER], qp[8], gp[8];
  bf16_t zp = 0;
  auto fetch = [&](int item) __attribute__((always_inline)) {
    const int bh = item / Tq, i = item - bh * Tq, b_ = bh / H, h_ = bh - b_ * H;
    const bf16_t* hz = HZ + (size_t)item * HZ_ELEMS;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint4 got = *(const uint4*)(hz + (size_t)(u * NT + t) * 8);
      hzp[u] = got;
    }
    zp = hz[D * D + (t & 127)];
    const long long n = min(i * BQ + nl, N - 1);
    const bf16_t* qrow = q + b_ * lq.sb + h_ * lq.sh + n * lq.sn + 8 * hf;
    const bf16_t* drow = dout + b_ * ld.sb + h_ * ld.sh + n * ld.sn + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint4 a = *(const uint4*)(qrow + 16 * ks), b = *(const uint4*)(drow + 16 * ks);
      qp[ks] = a;
      gp[ks] = b;
    }
  };
  if (first < end) fetch(first);

  for (int item = first; item < end; ++item) {
    // ---- publish H_i and Z_i
    hold_sums();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = u * NT + t, ln = x & 63, ks = (x >> 6) & 7, ot = x >> 9;
      *(uint4*)(Hl + (32 * ot + (ln & 31)) * TP + (32 * (ks >> 1) + 16 * (ln >> 5) + 8 * (ks & 1)) * 2) = hzp[u];
    }
    if (t < 128) zv[t] = bf16_to_f32(zp);
    const int bh = item / Tq, i = item - bh * Tq;
    const int n = i * BQ + nl;
    const bool ok = n < N;
    const uint32_t keep = ok ? ~0u : 0u;
    uint4 af[8], gf[8], qs[8 / CS];   // qs: of the wavefront's share of the channels
    float av[64];                // a = phi(Q[n]) at channels 16 ks + 8 hf + kk  (index 8 ks + kk)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      unpack8(qp[ks], &av[8 * ks]);
      if (ks < 8 / CS) qs[ks] = pair_order(CS == 2 && ch ? qp[(8 - 8 / CS) + ks] : qp[ks]);
      gf[ks] = uint4{gp[ks].x & keep, gp[ks].y & keep, gp[ks].z & keep, gp[ks].w & keep};
    }
    lds_barrier();

    float qmax = 0.f, rsum = 1.0f;
    if constexpr (PHI == 0) softmax_stats(av, qmax, rsum);
    else {
#pragma unroll
      for (int e = 0; e < 64; ++e) av[e] = phi_value<PHI>(av[e], 0.f, 1.0f);
    }
    if (!ok) rsum = 0.f;         // rows beyond the sequence take no part in dH, dZ, dW
    float den = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        av[8 * ks + kk] *= rsum;
        den += av[8 * ks + kk] * zv[16 * ks + 8 * hf + kk];
      }
      af[ks] = pack8(&av[8 * ks]);
      if (CS == 1 || (ks >> 2) == ch) *(uint4*)(Al + nl * TP + (16 * ks + 8 * hf) * 2) = af[ks];
    }
    den += partner_f32(den);
    const float rden = den > 0.f ? 1.0f / den : 0.f;

    // numT[o][n] = sum_c H[c][o] a[n][c]  ->  O^l;   glT[c'][n] = sum_r W[r][c'] dO[n][r]
    // (of the wavefront's own output tiles)
    v16f ol[OT], gl[OT];
    // (here and below: the LDS operand reads of a tile are grouped ahead of its matrix products;
    // left alone the compiler issues each read right before its product and waits for it every time)
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) {
      uint4 ah[8];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) ah[ks] = n_op(Hl + 32 * (OT * ch + ot) * TP, l32, hf, ks);
      __builtin_amdgcn_sched_barrier(0);
      ol[ot] = v16f{};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) ol[ot] = mfma_bf16(ah[ks], af[ks], ol[ot]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) af[ks] = pair_order(gf[ks]);   // (a is not needed in registers any more)
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) {
      uint4 aw[8];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) aw[ks] = t_op(Wl + 32 * (ks >> 1) * TP, tr_off, OT * ch + ot, ks & 1);
      __builtin_amdgcn_sched_barrier(0);
      gl[ot] = v16f{};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) gl[ot] = mfma_bf16(aw[ks], af[ks], gl[ot]);
      __builtin_amdgcn_sched_barrier(0);
    }
    float dden = 0.f;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        ol[ot][r] *= rden;
        dden += gl[ot][r] * ol[ot][r];
        gl[ot][r] *= rden;       // dnum
      }
    dden += partner_f32(dden);
    if (CS == 2 && hf == 0) half_dden[ch * BQ + nl] = dden;
    uint4 olp[OT][2], dn[4][2];  // O^l (all that is used of it from here on: the dW product) and dnum, rounded to bf16
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        olp[ot][s] = acc_operand(ol[ot], s);
        const uint4 d = dn[ot][s] = acc_operand(gl[ot], s);
        unsigned char* dst = Dl + nl * TP + (32 * (OT * ch + ot) + 16 * s + 4 * hf) * 2;
        *(uint2*)dst = uint2{d.x, d.y};
        *(uint2*)(dst + 16) = uint2{d.z, d.w};
      }
    if constexpr (CS == 2) {
      lds_barrier();             // dnum and the halves' shares of dden are complete
      dden = half_dden[nl] + half_dden[BQ + nl];
#pragma unroll
      for (int ot = 0; ot < 4; ++ot)   // dnum of all channels
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const unsigned char* src = Dl + nl * TP + (32 * ot + 16 * s + 4 * hf) * 2;
          const uint2 lo = *(const uint2*)src, hi = *(const uint2*)(src + 16);
          dn[ot][s] = uint4{lo.x, lo.y, hi.x, hi.y};
        }
    }
    dden *= -rden;
    if (hf == 0 && ch == 0) dden_s[nl] = dden;

    // ---- d phi(Q) = dnum H^T + dden Z, then through the softmax
    v16f da[OT];
#pragma unroll
    for (int ct = 0; ct < OT; ++ct) {
      uint4 ah[8];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) ah[ks] = t_op(Hl + 32 * (ks >> 1) * TP, tr_off, OT * ch + ct, ks & 1);
      __builtin_amdgcn_sched_barrier(0);
      da[ct] = v16f{};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) da[ct] = mfma_bf16(ah[ks], dn[ks >> 1][ks & 1], da[ct]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // a at the accumulator's channels 32 ct + 8 g + 4 hf + e, formed again from Q's words
    float sdot = 0.f;
#pragma unroll
    for (int ct = 0; ct < OT; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint4& qq = qs[2 * ct + (g >> 1)];
        const uint32_t q0 = g & 1 ? qq.z : qq.x, q1 = g & 1 ? qq.w : qq.y;
        const float xq[4] = {bf16_lo(q0), bf16_hi(q0), bf16_lo(q1), bf16_hi(q1)};
        const float4 z4 = *(const float4*)(zv + 32 * (OT * ch + ct) + 8 * g + 4 * hf);
        const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          da[ct][4 * g + e] += zz[e] * dden;
          if constexpr (PHI == 0) sdot += phi_value<0>(xq[e], qmax, rsum) * da[ct][4 * g + e];
        }
      }
    sdot += partner_f32(sdot);
    if (CS == 2 && hf == 0) half_sdot[ch * BQ + nl] = sdot;
    lds_barrier();               // every wavefront is done with H_i and Z_i; a, dnum, dden and the halves' shares of sdot are complete
    if constexpr (CS == 2) sdot = half_sdot[nl] + half_sdot[BQ + nl];
    asm volatile("" : "+v"(qmax));  // (a is formed once more below, not kept in 64 registers)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      if (CS == 1 || (ks >> 2) == ch) *(uint4*)(Hl + nl * TP + (16 * ks + 8 * hf) * 2) = gf[ks];
    if (ok) {
      float* drow = dq_lin + ((size_t)bh * N + n) * D;   // (the library's own tensor)
#pragma unroll
      for (int ct = 0; ct < OT; ++ct)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint4& qq = qs[2 * ct + (g >> 1)];
          const uint32_t q0 = g & 1 ? qq.z : qq.x, q1 = g & 1 ? qq.w : qq.y;
          const float xq[4] = {bf16_lo(q0), bf16_hi(q0), bf16_lo(q1), bf16_hi(q1)};
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            o[e] = phi_backward<PHI>(xq[e], phi_value<PHI>(xq[e], qmax, rsum), da[ct][4 * g + e], sdot);
          *(float4*)(drow + 32 * (OT * ch + ct) + 8 * g + 4 * hf) = float4{o[0], o[1], o[2], o[3]};
        }
    }

    // ---- dH_i^T[o][c] = sum_n dnum[n][o] a[n][c], dZ_i[c] = sum_n a[n][c] dden[n]
    hold_sums();
    // the next item: requested here, where the registers have room for it, used after the sections below
    __builtin_amdgcn_sched_barrier(0);
    fetch(min(item + 1, end - 1));
    __builtin_amdgcn_sched_barrier(0);
    bf16_t* dst = dHZ + (size_t)item * HZ_ELEMS;
    // (the store offsets below are formed from a value the compiler cannot see through: as loop
    // invariants they were kept in scratch memory, and each reload made its store wait for the one before)
    int lane_o = l32;
    asm volatile("" : "+v"(lane_o));
    uint4 aa[BQ / 16];
#pragma unroll
    for (int ks = 0; ks < BQ / 16; ++ks) aa[ks] = t_op(Al + 32 * (ks >> 1) * TP, tr_off, w, ks & 1);
#pragma unroll
    for (int x = 0; x < TILES; ++x) {
      v16f acc = v16f{};
      uint4 bb[BQ / 16];
#pragma unroll
      for (int ks = 0; ks < BQ / 16; ++ks) bb[ks] = t_op(Dl + 32 * (ks >> 1) * TP, tr_off, x, ks & 1);
#pragma unroll
      for (int ks = 0; ks < BQ / 16; ++ks) acc = mfma_bf16(aa[ks], bb[ks], acc);
      __builtin_amdgcn_sched_barrier(0);
      // lane: o = 32 x + l32; registers: c = 32 w + 8 g + 4 hf + e
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(uint2*)(dst + hz_run_offset(32 * x + lane_o, 32 * w + 8 * g + 4 * hf)) =
            uint2{pack_bf16x2(acc[4 * g], acc[4 * g + 1]), pack_bf16x2(acc[4 * g + 2], acc[4 * g + 3])};
    }
    __builtin_amdgcn_sched_barrier(0);
    float dz[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    tile_sums<BQ * 16 / NT>(Al, t, dz, [&](int m) { return dden_s[m]; });
    tile_sums_finish(dz, red, lane, w);
    lds_barrier();               // a and dnum are consumed
    if (t < 128) {
      float s = red[t];
#pragma unroll
      for (int u = 1; u < NW; ++u) s += red[u * 128 + t];
      dst[D * D + t] = f32_to_bf16(s);
    }

    // ---- dW[r][c] += sum_n dO[n][r] O^l[n][c],  db[r] += sum_n dO[n][r]
    if (dW_part) {
#pragma unroll
      for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          unsigned char* dst_o = Al + nl * TP + (32 * (OT * ch + ot) + 16 * s + 4 * hf) * 2;
          *(uint2*)dst_o = uint2{olp[ot][s].x, olp[ot][s].y};
          *(uint2*)(dst_o + 16) = uint2{olp[ot][s].z, olp[ot][s].w};
        }
      lds_barrier();
      uint4 ag[BQ / 16];         // the row tile of dO^T: the A operand of all its column tiles
#pragma unroll
      for (int ks = 0; ks < BQ / 16; ++ks) ag[ks] = t_op(Hl + 32 * (ks >> 1) * TP, tr_off, w, ks & 1);
#pragma unroll
      for (int x = 0; x < TILES; ++x) {
        uint4 bo[BQ / 16];
#pragma unroll
        for (int ks = 0; ks < BQ / 16; ++ks) bo[ks] = t_op(Al + 32 * (ks >> 1) * TP, tr_off, x, ks & 1);
#pragma unroll
        for (int ks = 0; ks < BQ / 16; ++ks) dwacc[x] = mfma_bf16(ag[ks], bo[ks], dwacc[x]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (db_part) tile_sums<BQ * 16 / NT>(Hl, t, dbacc, [](int) { return 1.0f; });
    lds_barrier();               // every tile is consumed
  }
  // This workgroup's share of dW and db goes to its own slice; reduce_block adds the
  // slices in a fixed order, so the sums do not depend on which workgroup finishes first.
  if (dW_part) {
    float* mine = dW_part + (size_t)blockIdx.x * (D * D);
#pragma unroll
    for (int x = 0; x < TILES; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        mine[(32 * w + 8 * (r >> 2) + 4 * hf + (r & 3)) * D + 32 * x + l32] = dwacc[x][r];
  }
  if (db_part) {
    tile_sums_finish(dbacc, red, lane, w);
    lds_barrier();
    if (t < 128) {
      float s = red[t];
#pragma unroll
      for (int u = 1; u < NW; ++u) s += red[u * 128 + t];
      db_part[(size_t)blockIdx.x * D + t] = s;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// One workgroup per compute unit at most: the partial sums' buffer is sized by it.
constexpr int LIN_Q_WORKGROUPS = 256;
static int lin_q_grid(const Problem& p) { return (int)std::min<long long>(LIN_Q_WORKGROUPS, (long long)p.BH * p.Tq); }
size_t bwd_lin_q_partial_bytes(const Problem& p) { return (size_t)lin_q_grid(p) * (D * D + D) * 4; }

template <int PHI>
static int launch_bwd_lin_q_phi(const Problem& p, const void* q, const void* dout, const bf16_t* HZ, const bf16_t* proj_w,
                                float* dq_lin, bf16_t* dHZ, float* dW, float* db, float* partials, ReduceArgs* reduce, hipStream_t stream) {
  constexpr int LDS4 = 4 * 128 * TP + (2 + 4) * 128 * 4, LDS2 = (2 * 128 + 2 * 64) * TP + (2 + 4) * 128 * 4 + 2 * 2 * 64 * 4;
  static const bool ok =
      hipFuncSetAttribute((const void*)bwd_lin_q_kernel<4, 1, PHI>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS4) == hipSuccess &&
      hipFuncSetAttribute((const void*)bwd_lin_q_kernel<2, 2, PHI>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS2) == hipSuccess;
  if (!ok) return -1;
  // per-workgroup partial sums: dW slices first, then db slices
  const int n_part = lin_q_grid(p);
  float* dW_part = dW ? partials : nullptr;
  float* db_part = db ? partials + (size_t)n_part * D * D : nullptr;
#define SLA_LIN_Q(TT, CS, LDS) bwd_lin_q_kernel<TT, CS, PHI><<<(unsigned)n_part, TT * CS * 64, LDS, stream>>>( \
      (const bf16_t*)q, (const bf16_t*)dout, HZ, proj_w, dq_lin, dHZ, dW_part, db_part, p.N, p.Tq, p.BH * p.Tq, p.H, p.lq, p.ld)
  if (p.block_q == 128) SLA_LIN_Q(4, 1, LDS4); else SLA_LIN_Q(2, 2, LDS2);
#undef SLA_LIN_Q
  *reduce = ReduceArgs{dW_part, db_part, n_part, dW, db};
  return 0;
}

int launch_bwd_lin_q(const Problem& p, const void* q, const void* dout, const bf16_t* HZ, const bf16_t* proj_w,
                     int phi_kind, float* dq_lin, bf16_t* dHZ, float* dW, float* db, float* partials, ReduceArgs* reduce, hipStream_t stream) {
  if (phi_kind == 0) return launch_bwd_lin_q_phi<0>(p, q, dout, HZ, proj_w, dq_lin, dHZ, dW, db, partials, reduce, stream);
  if (phi_kind == 1) return launch_bwd_lin_q_phi<1>(p, q, dout, HZ, proj_w, dq_lin, dHZ, dW, db, partials, reduce, stream);
  return launch_bwd_lin_q_phi<2>(p, q, dout, HZ, proj_w, dq_lin, dHZ, dW, db, partials, reduce, stream);
}

}  // namespace sla
