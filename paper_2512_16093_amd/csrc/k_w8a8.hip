// W8A8 Linear layer for gfx950: block-wise (128 x 128) INT8 quantisation of weights and
// activations and their product on the INT8 matrix units (Section 1.1, fourth technique;
// Section 1.3, "Linear layer quantization"; the formula is stated in include/w8a8.h).
//
// Operand order.  A quantised matrix A8[RP][K] (RP = rows padded to whole tiles, K a multiple
// of 128) is stored as 16-byte chunks
//     chunk ((kb * RT + rt) * 4 + ks) * 64 + lane,   RT = RP / 32,
// holding A8[32 rt + lane % 32][128 kb + 32 ks + 16 (lane / 32) + 0..15]: exactly what lane
// `lane` feeds to v_mfma_i32_32x32x32_i8 for row tile rt and contraction step ks of feature
// block kb.  Everything a workgroup needs of one feature block is then contiguous (4 KiB per
// row tile, consecutive row tiles adjacent), so operands move with straight 16-byte-per-lane
// copies.  Scales: s[kb * RB + rb], RB = RP / 128.  Rows past the end hold zero codes.
//
// Kernels
//   w8a8_quantize_kernel   one workgroup per 128 x 128 block: amax, scale, codes through LDS
//                          into operand order.  HBM-bound (reads 2 bytes, writes 1 per element).
//   w8a8_gemm_kernel       workgroup tile 256 tokens x 128 outputs, four wavefronts of 64 x 128.
//                          The weight tile of a feature block (16 KiB) is staged in LDS by
//                          asynchronous copies, three stages deep; a wavefront's activation
//                          operands (8 KiB per feature block) go from global memory straight to
//                          registers, one feature block ahead.  INT8 MFMA bound.
//   w8a8_gemm_splitk_kernel  small workgroup tiles whose wavefronts split the contraction, for calls that do not
//                          give every compute unit a 256 x 128 tile.
#include "common.h"

namespace sla {

constexpr int QB = 128;                      // quantisation block edge
constexpr int W8_WG_M = 256, W8_WG_N = 128;  // workgroup tile of the product
// The integer accumulators start from the bit pattern of the float 1 / (2 pi), which the MFMA
// takes as its C operand: a finished accumulator, reinterpreted as fp32, is then exactly
// W8_C0 + s * 2^-26 for every block sum |s| <= 127 * 127 * 128 (the pattern stays inside the
// binade [1/8, 1/4)), so scaling and accumulating a block is ONE fma per element, with no
// int -> float conversion.  The constant's share must stay small next to the sums it rides on
// (fp32 rounds at the magnitude of the running total): the weight codes of ODD feature blocks
// are stored negated and their blocks scaled by -s_X s_W, which leaves the products' share
// unchanged and makes the constants alternate in sign; what is left of them, W8_C0 * (signed
// sum of the scales), is uniform over a wavefront's tile and is taken out at the end.
constexpr int W8_BIAS_I = 0x3E22F983;
constexpr float W8_C0 = 0.15915494f;         // the float with that bit pattern
constexpr float W8_STEP_INV = 67108864.0f;   // 2^26

__host__ __device__ inline size_t w8_chunk(int kb, int RT, int rt, int ks) {
  return (((size_t)kb * RT + rt) * 4 + ks) * 64;  // index of the first of the 64 chunks (lanes)
}

// ---------------------------------------------------------------------------
// Quantisation of one 128 x 128 block per workgroup.  Thread t: columns 8 (t % 16) .. +7 of
// rows t / 16 + 16 i, i = 0..7.
// ---------------------------------------------------------------------------
// negate_odd (weights): the codes of odd feature blocks are stored negated (see W8_BIAS_I).
// STREAM: the input is read past the caches (it exceeds what the memory-side cache keeps beside the codes, which the
// product reads next).
template <bool STREAM>
__global__ void __launch_bounds__(256) w8a8_quantize_kernel(const bf16_t* __restrict__ a, int R, int K, int RP,
                                                            int negate_odd, int8_t* __restrict__ codes,
                                                            float* __restrict__ scales) {
  __shared__ uint4 blk[QB * QB / 16];
  __shared__ float wave_amax[4];
  const int KB = K / QB, RB = RP / QB, RT = RP / 32;
  const int rb = blockIdx.x / KB, kb = blockIdx.x % KB;
  const int t = threadIdx.x, cg = t & 15, r0 = t >> 4, lane = t & 63, w = t >> 6;
  uint4 x[8];
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = rb * QB + r0 + 16 * i;
    x[i] = make_uint4(0, 0, 0, 0);
    if (row < R) {
      const v4i* src = (const v4i*)(a + (size_t)row * K + kb * QB + cg * 8);
      x[i] = __builtin_bit_cast(uint4, STREAM ? __builtin_nontemporal_load(src) : *src);
    }
    const uint32_t wd[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(wd[e])), fabsf(bf16_hi(wd[e]))));
  }
  for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
  if (lane == 0) wave_amax[w] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(wave_amax[0], wave_amax[1]), fmaxf(wave_amax[2], wave_amax[3]));
  const float s = amax > 0.f ? amax / 127.0f : 1.0f;
  if (t == 0) scales[kb * RB + rb] = s;
  // codes = the correctly rounded quotient 127 x / amax, rounded to the nearest integer with ties to even
  // (int8_code_word_exact: exact ties stay ties -- with 16-bit inputs they are common, x = amax / 2 is one);
  // the two's-complement low byte of the returned word is the code; |x / s| <= 127.
  const CodeScale cs = code_scale(amax, 127.0f);
  const float sgn = (negate_odd && (kb & 1)) ? -1.0f : 1.0f;
  unsigned char* out = (unsigned char*)blk;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t wd[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
    uint32_t b[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      b[2 * e] = int8_code_word_exact(sgn * bf16_lo(wd[e]), cs);
      b[2 * e + 1] = int8_code_word_exact(sgn * bf16_hi(wd[e]), cs);
    }
    const uint32_t lo = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u),
                                              __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), 0x05040100u);
    const uint32_t hi = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[7], b[6], 0x0c0c0400u),
                                              __builtin_amdgcn_perm(b[5], b[4], 0x0c0c0400u), 0x05040100u);
    const int rl = r0 + 16 * i;  // row within the block
    const int off = (((rl >> 5) * 4 + (cg >> 2)) * 64 + (rl & 31) + 32 * ((cg >> 1) & 1)) * 16 + 8 * (cg & 1);
    *(uint2*)(out + off) = make_uint2(lo, hi);
  }
  __syncthreads();
  // the block's four row tiles x four steps are one contiguous 16 KiB in operand order
  uint4* dst = (uint4*)codes + w8_chunk(kb, RT, 4 * rb, 0);
#pragma unroll
  for (int u = 0; u < 4; ++u) dst[u * 256 + t] = blk[u * 256 + t];
}

// Plain-layout copies of codes and scales (tests only).
__global__ void w8a8_unpack_kernel(const int8_t* __restrict__ frag, const float* __restrict__ s, int R, int K, int RP,
                                   int negate_odd, int8_t* __restrict__ codes, float* __restrict__ scales) {
  const int KB = K / QB, RB = RP / QB, RT = RP / 32;
  const size_t total = (size_t)R * K;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int r = (int)(i / K), k = (int)(i % K);
    const int kb = k / QB, ks = (k % QB) / 32, half = (k % 32) / 16, byte = k % 16;
    const int8_t c = frag[(w8_chunk(kb, RT, r / 32, ks) + (r % 32) + 32 * half) * 16 + byte];
    if (codes) codes[i] = (negate_odd && (kb & 1)) ? (int8_t)-c : c;
  }
  const int rbn = (R + QB - 1) / QB;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; scales && i < (size_t)rbn * KB;
       i += (size_t)gridDim.x * blockDim.x)
    scales[i] = s[(i % KB) * RB + i / KB];
}

// ---------------------------------------------------------------------------
// The product.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* w8_lds_ptr_t;
// Asynchronous 16-bytes-per-lane copy global -> LDS (lane l reads base + voff, the data lands at
// lds + 16 l), issued from inline assembly so that the compiler does not make every LDS read
// wait for all copies in flight; the pipeline waits for them by explicit counts.
__device__ __forceinline__ void w8_copy16(const void* base, unsigned voff, const void* lds) {
  const unsigned lds_addr = (unsigned)(uintptr_t)(w8_lds_ptr_t)lds;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
               :
               : "s"(base), "v"(voff), "s"(lds_addr)
               : "memory", "m0");
}
__device__ __forceinline__ void w8_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The first product of a chain takes the pattern W8_BIAS_I as an inline constant (0.15915494 is
// the assembler's spelling of 1 / (2 pi)); the compiler would keep the constant in sixteen
// registers instead.  Every product of a chain is an assembly statement whose accumulator is ONE
// in/out operand, so the chain accumulates in place by construction (destination = C operand,
// the case the hardware interlocks) whatever registers are allocated, and each product still
// takes its operands as they arrive.  The compiler does not know the statements hold
// matrix products and adds no wait states before a vector instruction that reads the result, so
// the data flow itself keeps every reader a whole chain (four dependent products, > 100 cycles)
// behind: a chain's result may only be read after it has been handed through the SECOND product
// of the next chain as `carry` (an in/out operand the statement does not touch; that product
// cannot issue before the next chain's first one has finished, 64 cycles after the carried
// chain's last one was issued), or, after the loop, through a statement of explicit wait states.
__device__ __forceinline__ v16i w8_chain(const v4i (&b)[4], const v4i (&ar)[4], v16i& carry) {
  v16i acc;
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 0.15915494" : "=&v"(acc) : "v"(b[0]), "v"(ar[0]));
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %2, %3, %0" : "+v"(acc), "+v"(carry) : "v"(b[1]), "v"(ar[1]));
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc) : "v"(b[2]), "v"(ar[2]));
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc) : "v"(b[3]), "v"(ar[3]));
  return acc;
}
// The wait states a vector read of a matrix product's result needs, where no later chain keeps the distance.
#define W8_READ_WAIT "s_nop 7\n\ts_nop 7\n\ts_nop 3"
__device__ __forceinline__ void w8_scale_in(const v16i& acc, float sc, v16f& f) {
#pragma unroll
  for (int e = 0; e < 16; ++e) f[e] = __builtin_fmaf(__int_as_float(acc[e]), sc, f[e]);
}

constexpr int W8_DEAL_MT = 64;  // token tiles from which whole ones are dealt to the XCDs
constexpr int W8_EPI_STRIDE = W8_WG_N * 2 + 16;  // bytes per staged output row

__global__ void __launch_bounds__(256, 2) w8a8_gemm_kernel(
    const int8_t* __restrict__ x8, const float* __restrict__ sx, const int8_t* __restrict__ w8,
    const float* __restrict__ sw, const bf16_t* __restrict__ bias, bf16_t* __restrict__ y, int M, int N, int K,
    int RTx, int RBx, int RTw, int RBw, int MT, int NT) {
  __shared__ uint4 bst[3][QB * W8_WG_N / 16];  // three stages of a 128-feature x 128-output weight tile
  static_assert(4 * 32 * W8_EPI_STRIDE <= (int)sizeof(uint4) * 3 * QB * W8_WG_N / 16, "output staging fits the stages");
  // Workgroup ids are dealt round-robin over the 8 XCDs.  An XCD walks its tiles in patch order: bands of 8 token
  // tiles, in a band groups of 8 output tiles, output tiles fastest (ragged bands and groups are just smaller).  64
  // consecutive workgroups -- what its 32 compute units hold at a time -- so form a patch of 8 x 8 tiles that
  // walks the feature blocks at the same pace, and each activation and weight tile of a feature block is fetched
  // into that L2 once for eight users.  Its share: of many token tiles, every eighth (x, x + 8, ...: the XCDs then
  // read adjacent ones at a time; 75600 tokens x 5120 -> 5120 2.151 ms against 2.169 ms for runs); of few, where
  // whole token tiles would not divide evenly (1024 tokens, 4 of them, left four XCDs idle: 5120 -> 13824 153
  // against 86 us), an eighth of the tiles in patch order, equal to within one.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const bool deal = MT >= W8_DEAL_MT;
  const int per = (MT * NT + 7) >> 3, first = deal ? 0 : xcd * per;
  const int rows = deal ? (MT - xcd + 7) >> 3 : MT;   // token tiles of the walk
  if (slot >= (deal ? rows * NT : min(per, MT * NT - first))) return;
  const int idx = first + slot, band = idx / (8 * NT), in_band = idx - band * 8 * NT, band_rows = min(8, rows - 8 * band);
  const int grp = in_band / (8 * band_rows), in_grp = in_band - grp * 8 * band_rows;
  const int cols = min(8, NT - 8 * grp), row = 8 * band + in_grp / cols;
  const int mt = __builtin_amdgcn_readfirstlane(deal ? 8 * row + xcd : row);
  const int nt = __builtin_amdgcn_readfirstlane(8 * grp + in_grp % cols);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  const int KB = K / QB;
  const int rt0 = mt * (W8_WG_M / 32) + 2 * w;  // this wavefront's two row tiles (64 tokens)
  const int rb = mt * 2 + (w >> 1);             // and their quantisation block row
  const unsigned char* xa = (const unsigned char*)x8 + (size_t)rt0 * 4096 + (size_t)lane * 16;
  const size_t xkb = (size_t)RTx * 4096;        // bytes from one feature block to the next
  const unsigned char* wb = (const unsigned char*)w8 + (size_t)(4 * nt) * 4096;
  const size_t wkb = (size_t)RTw * 4096;

  auto fetch_b = [&](int kb) {  // 16 KiB weight tile of feature block kb -> its stage; four 1 KiB pieces per wavefront
    const unsigned char* src = wb + (size_t)kb * wkb;
    unsigned char* dst = (unsigned char*)bst[kb % 3];
#pragma unroll
    for (int u = 0; u < 4; ++u) w8_copy16(src, (unsigned)((w * 4 + u) * 1024 + lane * 16), dst + (w * 4 + u) * 1024);
  };

  auto load_half = [&](int kb, int rtl, v4i (&a)[2][4]) __attribute__((always_inline)) {  // one of the two row tiles
    const unsigned char* src = xa + (size_t)kb * xkb;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[rtl][ks] = *(const v4i*)(src + (rtl * 4 + ks) * 1024);
  };
  v16f facc[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) facc[r][c] = v16f{};
  v16i bias16;  // (only the idle value of `pend` below; the chains take the pattern as an inline constant)
#pragma unroll
  for (int e = 0; e < 16; ++e) bias16[e] = W8_BIAS_I;
  float csum = 0.f;                 // scales whose constant share is still inside facc

  v4i a0[2][4], a1[2][4];  // this wavefront's activation operands of the current and the next feature block

  // One feature block: products against the staged weight tile, then one fma per element.  The
  // product is taken transposed (weights as the A operand) so that a lane owns ONE token and runs
  // of four consecutive outputs.
  // The chains (4 output tiles x 2 token tiles per feature block) run back to back on the matrix
  // pipe, each with the fmas of the chain before it interleaved for the vector ALU -- across
  // feature blocks too: the last chain of a block is scaled in next to the first chain of the
  // next one.  Scheduling barriers and register anchors keep the compiler from stretching that
  // window (and the registers it needs).
  v16i pend = bias16;   // finished chain still to be scaled in (token tile 1, output tile 3); none yet: s = 0
  float pend_sc = 0.f;
  auto compute = [&](int kb, const v4i (&a)[2][4], auto more) __attribute__((always_inline)) {
    const float mag = sx[(size_t)kb * RBx + rb] * sw[(size_t)kb * RBw + nt] * W8_STEP_INV;
    const float sc = (kb & 1) ? -mag : mag;
    const uint4* st = bst[kb % 3];
    v16i acc0;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      v4i b[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        union { uint4 u; v4i v; } x;
        x.u = st[(ct * 4 + ks) * 64 + lane];
        b[ks] = x.v;
      }
      acc0 = w8_chain(b, a[0], pend);       // (from here on the previous chain's result may be read)
      v16f& ftile = facc[1][(ct + 3) & 3];
      w8_scale_in(pend, pend_sc, ftile);
      asm volatile("" : "+v"(ftile) : : "memory");  // (the fmas stay in this window)
      asm volatile("" : "+v"(acc0) : : "memory");
      __builtin_amdgcn_sched_barrier(0);
      {
        v16i fresh = w8_chain(b, a[1], acc0);
        pend = fresh;
      }
      pend_sc = sc;
      w8_scale_in(acc0, sc, facc[0][ct]);
      asm volatile("" : "+v"(facc[0][ct]) : : "memory");
      asm volatile("" : "+v"(pend) : : "memory");
      more(ct);
      __builtin_amdgcn_sched_barrier(0);
    }
    csum += sc;
  };

  // Pipeline.  The weight tiles run two feature blocks ahead of the products (three LDS stages),
  // the activation operands one block ahead (two register sets).  At the top of step kb
  // everything this wavefront has requested is waited for -- all of it was requested at least
  // half a block earlier; the barrier then publishes everybody's share of stage kb and retires
  // stage kb - 1, which the copy of block kb + 2 overwrites.  The activations are requested behind
  // the first and the second quarter of the products, not in one burst behind the barrier: the memory path
  // has to deliver 47 of its 64 bytes per clock and compute unit at full matrix rate.  With that and the bias read
  // at once (below) the layer went from 2129 to 1977 us at 75600 x 5120 -> 5120, from 573 to 488 at 32760 x 1536 -> 8960; with
  // no operand loads at all (timing only) it would be 1610 us.  Requests ahead into L2 made it slower (2040 us): it is
  // not the latency.  (The last step requests its own block's activations once more, 8 KiB per wavefront that nobody
  // reads: the schedule stays the same for every step.)
  fetch_b(0);
  if (KB > 1) fetch_b(1);
  load_half(0, 0, a0);
  load_half(0, 1, a0);
#define W8_STEP(KBI, ACUR, ANEXT)                       \
  {                                                     \
    const int kb_ = (KBI);                              \
    __builtin_amdgcn_s_waitcnt(0x0F70); /* vmcnt(0) */  \
    w8_barrier();                                       \
    if (kb_ + 2 < KB) fetch_b(kb_ + 2);                 \
    compute(kb_, ACUR, [&](int ct) __attribute__((always_inline)) { if (ct < 2) load_half(min(kb_ + 1, KB - 1), ct, ANEXT); }); \
  }
  {
    int kb = 0;
    for (; kb + 2 <= KB; kb += 2) {
      W8_STEP(kb, a0, a1)
      W8_STEP(kb + 1, a1, a0)
    }
    if (kb < KB) W8_STEP(kb, a0, a1)
  }
#undef W8_STEP
  asm volatile(W8_READ_WAIT : "+v"(pend));
  w8_scale_in(pend, pend_sc, facc[1][3]);

  // Epilogue: constant share out, bias in, bf16, through LDS so that rows leave as 256 contiguous
  // bytes.  Lane = token 32 rt + l32 of this wavefront; registers 4 g .. 4 g + 3 of tile ct =
  // outputs 32 ct + 8 g + 4 hf + 0..3.
  w8_barrier();  // every wavefront is done with the stages
  unsigned char* my = (unsigned char*)bst + w * (32 * W8_EPI_STRIDE);
  const int n0 = nt * W8_WG_N;
  uint2 bw[4][4];   // (all sixteen at once: one by one behind a test for a bias each waited for memory by itself)
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int g = 0; g < 4; ++g) bw[ct][g] = make_uint2(0u, 0u);
  if (bias) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) bw[ct][g] = *(const uint2*)(bias + n0 + 32 * ct + 8 * g + 4 * hf);
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint2 b4 = bw[ct][g];
        const float bv[4] = {bf16_lo(b4.x), bf16_hi(b4.x), bf16_lo(b4.y), bf16_hi(b4.y)};
        const v16f& f = facc[r][ct];
        auto sum = [&](float x) __attribute__((always_inline)) { return __builtin_fmaf(-W8_C0, csum, x); };   // (the constants' share, not rounded by itself)
        *(uint2*)(my + l32 * W8_EPI_STRIDE + (32 * ct + 8 * g + 4 * hf) * 2) =
            make_uint2(pack_bf16x2(sum(f[4 * g]) + bv[0], sum(f[4 * g + 1]) + bv[1]),
                       pack_bf16x2(sum(f[4 * g + 2]) + bv[2], sum(f[4 * g + 3]) + bv[3]));
      }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront's staging writes are done
    asm volatile("" ::: "memory");
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int row = it * 4 + (lane >> 4), part = lane & 15;
      const int m = mt * W8_WG_M + 64 * w + 32 * r + row;
      const v4i v = *(const v4i*)(my + row * W8_EPI_STRIDE + part * 16);
      // (past the caches: the results would push the operands out of them, 75600 x 1536 -> 1536 314 -> 286 us,
      // 32760 x 1536 -> 8960 678 -> 645 us for the layer)
      if (m < M) __builtin_nontemporal_store(v, (v4i*)(y + (size_t)m * N + n0 + part * 8));
    }
    asm volatile("" ::: "memory");
  }
}

// ---------------------------------------------------------------------------
// The product for calls with few tokens or few outputs, where 256 x 128 tiles leave compute units without work
// and every workgroup walks the whole contraction alone (512 x 5120 -> 5120: 80 tiles, 40 feature blocks each).
// Workgroup tile (32 RT) tokens x (32 CT) outputs; its KS wavefronts split the CONTRACTION: each runs the whole
// tile over a contiguous run of feature blocks (contiguous, so that the constants still alternate in sign from
// block to block) and the partial sums meet in LDS in a fixed order.
// Both operands go from memory straight to registers: they are in operand order, so a fragment is one contiguous
// KiB, nothing is shared between the wavefronts, and there is no barrier in the loop.  A fragment is requested
// again for the next feature block right behind the last product that reads it, half a block or more ahead of its
// next use.  Bound by the CU's 64 bytes per clock from L2 (16 KiB per 16 products at RT = CT = 2).
// ---------------------------------------------------------------------------
template <int RT, int CT, int KS>
__global__ void __launch_bounds__(64 * KS, 2) w8a8_gemm_splitk_kernel(
    const int8_t* __restrict__ x8, const float* __restrict__ sx, const int8_t* __restrict__ w8,
    const float* __restrict__ sw, const bf16_t* __restrict__ bias, bf16_t* __restrict__ y, int M, int N, int K,
    int RTx, int RBx, int RTw, int RBw, int MT, int NT) {
  constexpr int PITCH = 36;  // floats per staged row of 32 outputs (16-byte rows, skewed banks)
  __shared__ __attribute__((aligned(16))) float part[KS][32 * RT][PITCH];
  // XCD x takes a contiguous eighth of the tiles, along the smaller operand fastest: of the larger one a tile is then
  // fetched into one L2 only (always along the tokens: 30000 x 8960 -> 256 156 us, now 115; 10000 x 256 -> 1536 17.6, now
  // 15.5; in large tiles they were 121 and 16.5 before there was a choice).
  const int per = (MT * NT + 7) >> 3, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int idx = __builtin_amdgcn_readfirstlane(xcd * per + slot);
  if ((int)(blockIdx.x >> 3) >= per || idx >= MT * NT) return;
  const bool tokens_fastest = M <= N;
  const int major = __builtin_amdgcn_readfirstlane(idx / (tokens_fastest ? MT : NT)), minor = idx - major * (tokens_fastest ? MT : NT);
  const int nt = tokens_fastest ? major : minor, mt = tokens_fastest ? minor : major;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  const int KB = K / QB;
  const int kb0 = KB * w / KS, kb1 = KB * (w + 1) / KS;  // this wavefront's feature blocks (none: an empty run)
  const int rb = mt * RT / 4, nb = nt * CT / 4;          // quantisation blocks of the tile
  const unsigned char* xa = (const unsigned char*)x8 + (size_t)(mt * RT) * 4096 + (size_t)lane * 16;
  const unsigned char* wb = (const unsigned char*)w8 + (size_t)(nt * CT) * 4096 + (size_t)lane * 16;
  const size_t xkb = (size_t)RTx * 4096, wkb = (size_t)RTw * 4096;

  // Where the contraction is split, a run's sums start from minus the constant share of its first block: every other
  // block then adds at the sums' own magnitude whatever the run's first block and length, and a sum is rounded at the
  // constants' magnitude no more often than in one walk.  (Started from zero, runs of odd lengths were rounded up to twice
  // as often: 200 x 384 -> 8192, 17 % of the outputs were not the rounded exact sum; in one walk 12 %, like this 10 %.)
  const float mag0 = kb0 < kb1 ? sx[(size_t)kb0 * RBx + rb] * sw[(size_t)kb0 * RBw + nb] * W8_STEP_INV : 0.f;
  const float base = KS == 1 ? 0.f : W8_C0 * ((kb0 & 1) ? mag0 : -mag0);
  v16f facc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) facc[r][c][e] = base;
  float csum = 0.f;
  if (kb0 < kb1) {
    v4i a[RT][4], b[CT][4];
    auto load_frag = [&](const unsigned char* tile, v4i (&f)[4]) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) f[ks] = *(const v4i*)(tile + ks * 1024);
    };
    auto block_scale = [&](int kb) { return sx[(size_t)kb * RBx + rb] * sw[(size_t)kb * RBw + nb] * W8_STEP_INV; };
#pragma unroll
    for (int c = 0; c < CT; ++c) load_frag(wb + (size_t)kb0 * wkb + c * 4096, b[c]);
#pragma unroll
    for (int r = 0; r < RT; ++r) load_frag(xa + (size_t)kb0 * xkb + r * 4096, a[r]);
    float mag = mag0;
    v16i pend;              // finished chain still to be scaled in; none yet: any finite pattern at scale 0
#pragma unroll
    for (int e = 0; e < 16; ++e) pend[e] = W8_BIAS_I;
    float pend_sc = 0.f;
    for (int kb = kb0; kb < kb1; ++kb) {
      const float sc = (kb & 1) ? -mag : mag;
      const int kn = min(kb + 1, kb1 - 1);   // (the last block is requested once more: the loop stays free of branches)
      mag = block_scale(kn);
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          v16i fresh = w8_chain(b[c], a[r], pend);   // (from here on the previous chain's result may be read)
          v16f& prev = r > 0 ? facc[r - 1][c] : facc[RT - 1][(c + CT - 1) % CT];
          w8_scale_in(pend, pend_sc, prev);
          asm volatile("" : "+v"(prev) : : "memory");
          asm volatile("" : "+v"(fresh) : : "memory");
          if (c == CT - 1) load_frag(xa + (size_t)kn * xkb + r * 4096, a[r]);
          if (r == RT - 1) load_frag(wb + (size_t)kn * wkb + c * 4096, b[c]);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (RT * CT == 1) {
            // (a lone chain per block cannot be carried over the loop's back edge without a copy, which would
            // read it too early: it is waited for and scaled in here, the other wavefronts fill the pipe)
            asm volatile(W8_READ_WAIT : "+v"(fresh));
            w8_scale_in(fresh, sc, facc[0][0]);
          } else {
            pend = fresh;
            pend_sc = sc;
          }
        }
      csum += sc;
    }
    if constexpr (RT * CT > 1) {
      asm volatile(W8_READ_WAIT : "+v"(pend));
      w8_scale_in(pend, pend_sc, facc[RT - 1][CT - 1]);
    }
  }

  // Partial sums (constant share out) through LDS, one column tile at a time; lane = token, registers
  // 4 g .. 4 g + 3 = outputs 8 g + 4 hf + 0..3.  Each thread then adds eight outputs of a token, in wavefront order.
  const float corr = __builtin_fmaf(W8_C0, csum, base);
  for (int c = 0; c < CT; ++c) {
    if (c > 0) __syncthreads();
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        v16f f = facc[r][0];
#pragma unroll
        for (int cc = 1; cc < CT; ++cc)
          if (c == cc) f = facc[r][cc];
        *(float4*)&part[w][32 * r + l32][8 * g + 4 * hf] =
            make_float4(f[4 * g] - corr, f[4 * g + 1] - corr, f[4 * g + 2] - corr, f[4 * g + 3] - corr);
      }
    __syncthreads();
    const int n0 = (nt * CT + c) * 32;
    for (int u = t; u < 32 * RT * 4; u += 64 * KS) {
      const int row = u >> 2, o = 8 * (u & 3), m = mt * 32 * RT + row;
      if (m >= M) continue;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = part[0][row][o + e];
#pragma unroll
      for (int p = 1; p < KS; ++p)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += part[p][row][o + e];
      if (bias) {
        const uint2 b0 = *(const uint2*)(bias + n0 + o), b1 = *(const uint2*)(bias + n0 + o + 4);
        v[0] += bf16_lo(b0.x); v[1] += bf16_hi(b0.x); v[2] += bf16_lo(b0.y); v[3] += bf16_hi(b0.y);
        v[4] += bf16_lo(b1.x); v[5] += bf16_hi(b1.x); v[6] += bf16_lo(b1.y); v[7] += bf16_hi(b1.y);
      }
      *(uint4*)(y + (size_t)m * N + n0 + o) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                        pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
  }
}

// The same with larger tiles, one wavefront per SIMD (the fp32 sums of a 64 x 160 tile alone take 160 registers): per product
// 0.7 KiB have to come from L2 instead of 1, and between 64 x 96 and 128 x 96 there is a tile that deals out in one round
// where 64 x 64 ones leave a last round nearly empty (512 x 5120 -> 5120: 256 tiles of 64 x 160, one per compute unit; of 64 x
// 64 there are 2.5).  The operands are held in accumulation registers, where the sums cannot be, the activations of a feature
// block requested a whole block ahead (two sets), a weight fragment behind its last product: with one set, half a block ahead,
// 512 x 5120 -> 5120 took 22.1 instead of 19.8 us.  Of a wavefront's 32.8 k cycles there (products alone: 12.8 k) 2.8 k pass
// until its first operands are requested, 3.0 k with its first pair of blocks, 20.7 k with the other four, 6.3 k while the
// sums go through LDS; 2590 a block, in which the products take 1280 and the compute unit gets 115 KB from L2, 44 bytes per
// clock of the 64 that the path carries.  Bound by no unit alone: by that path in the loop, by waiting around it.
// A tile's outputs may span two quantisation blocks (CT = 3, 5: two scales), and the last tile of a row may reach past N (its
// operands are then the last fragment's once more and nothing of it is stored).
// (w8_chain with both operands in accumulation registers; 0x3e22f983 is W8_BIAS_I, the same inline constant)
__device__ __forceinline__ v16i w8_chain_acc(const v4i (&b)[4], const v4i (&ar)[4], v16i& carry) {
  v16i acc;
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 0x3e22f983" : "=&v"(acc) : "a"(b[0]), "a"(ar[0]));
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %2, %3, %0" : "+v"(acc), "+v"(carry) : "a"(b[1]), "a"(ar[1]));
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc) : "a"(b[2]), "a"(ar[2]));
  asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc) : "a"(b[3]), "a"(ar[3]));
  return acc;
}
template <int RT, int CT, int KS>
__global__ void __launch_bounds__(64 * KS, 1) w8a8_gemm_wide_kernel(
    const int8_t* __restrict__ x8, const float* __restrict__ sx, const int8_t* __restrict__ w8,
    const float* __restrict__ sw, const bf16_t* __restrict__ bias, bf16_t* __restrict__ y, int M, int N, int K,
    int RTx, int RBx, int RTw, int RBw, int MT, int NT) {
  static_assert(CT <= 5 && (RT == 2 || RT == 4) && KS > 1, "a tile lies in one block of tokens and at most two of outputs");
  constexpr int PITCH = 36;  // floats per staged row of 32 outputs (16-byte rows, skewed banks)
  __shared__ __attribute__((aligned(16))) float part[2][KS][32 * RT][PITCH];
  const int per = (MT * NT + 7) >> 3, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;   // (dealt as above)
  const int idx = __builtin_amdgcn_readfirstlane(xcd * per + slot);
  if (slot >= per || idx >= MT * NT) return;
  const bool tokens_fastest = M <= N;
  const int major = __builtin_amdgcn_readfirstlane(idx / (tokens_fastest ? MT : NT)), minor = idx - major * (tokens_fastest ? MT : NT);
  const int nt = tokens_fastest ? major : minor, mt = tokens_fastest ? minor : major;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  const int KB = K / QB;
  // This wavefront's feature blocks, in pairs (the two sets of activations in turn): an odd last one is followed by a block
  // that does not exist, whose scale is zero.
  const int pairs = (KB + 1) >> 1, kb0 = 2 * (pairs * w / KS), kb1 = 2 * (pairs * (w + 1) / KS);
  const int ct0 = nt * CT, rb = mt * RT / 4, nb0 = ct0 >> 2, nb1 = min(nb0 + 1, RBw - 1);
  auto second = [&](int c) { return ((ct0 + c) >> 2) != nb0; };
  const unsigned char* xa = (const unsigned char*)x8 + (size_t)(mt * RT) * 4096 + (size_t)lane * 16;
  const unsigned char* wb = (const unsigned char*)w8 + (size_t)lane * 16;
  const size_t xkb = (size_t)RTx * 4096, wkb = (size_t)RTw * 4096;
  size_t wct[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) wct[c] = (size_t)min(ct0 + c, RTw - 1) * 4096;

  // (a run's sums start from minus the constant share of its first block: see above)
  auto mag_of = [&](int kb, int nb) { return sx[(size_t)kb * RBx + rb] * sw[(size_t)kb * RBw + nb] * W8_STEP_INV; };
  float mag[2] = {0.f, 0.f}, base[2] = {0.f, 0.f}, csum[2] = {0.f, 0.f};
  if (kb0 < kb1) {
    mag[0] = mag_of(kb0, nb0);
    mag[1] = mag_of(kb0, nb1);
#pragma unroll
    for (int u = 0; u < 2; ++u) base[u] = -W8_C0 * mag[u];   // (kb0 is even)
  }
  v16f facc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const float from = second(c) ? base[1] : base[0];
#pragma unroll
      for (int e = 0; e < 16; ++e) facc[r][c][e] = from;
    }
  if (kb0 < kb1) {
    v4i a0[RT][4], a1[RT][4], b[CT][4];
    auto load_frag = [&](const unsigned char* tile, v4i (&f)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) f[ks] = *(const v4i*)(tile + ks * 1024);
    };
#pragma unroll
    for (int c = 0; c < CT; ++c) load_frag(wb + (size_t)kb0 * wkb + wct[c], b[c]);
    v16i pend;              // finished chain still to be scaled in; none yet: any finite pattern at scale 0
#pragma unroll
    for (int e = 0; e < 16; ++e) pend[e] = W8_BIAS_I;
    float pend_sc = 0.f;
    // (an even number of chains, so that the two accumulators end a step where they began it: a copy would read one too early)
    static_assert(RT * CT % 2 == 0, "two accumulators in turn");
    auto step = [&](int kb, const v4i (&a)[RT][4], v4i (&an)[RT][4]) __attribute__((always_inline)) {
      float sc[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) sc[u] = kb < KB ? ((kb & 1) ? -mag[u] : mag[u]) : 0.f;
      const int kn = min(kb + 1, KB - 1);   // (past the end the last block once more: the loop stays free of branches)
      mag[0] = mag_of(kn, nb0);
      mag[1] = mag_of(kn, nb1);
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          v16i fresh = w8_chain_acc(b[c], a[r], pend);   // (from here on the previous chain's result may be read)
          v16f& prev = r > 0 ? facc[r - 1][c] : facc[RT - 1][(c + CT - 1) % CT];
          w8_scale_in(pend, pend_sc, prev);
          asm volatile("" : "+v"(prev) : : "memory");
          asm volatile("" : "+v"(fresh) : : "memory");
          if (c == 0) load_frag(xa + (size_t)kn * xkb + r * 4096, an[r]);
          if (r == RT - 1) load_frag(wb + (size_t)kn * wkb + wct[c], b[c]);
          __builtin_amdgcn_sched_barrier(0);
          pend = fresh;
          pend_sc = second(c) ? sc[1] : sc[0];
        }
      csum[0] += sc[0];
      csum[1] += sc[1];
    };
#pragma unroll
    for (int r = 0; r < RT; ++r) load_frag(xa + (size_t)kb0 * xkb + r * 4096, a0[r]);
    for (int kb = kb0; kb < kb1; kb += 2) {
      step(kb, a0, a1);
      step(kb + 1, a1, a0);
    }
    asm volatile(W8_READ_WAIT : "+v"(pend));
    w8_scale_in(pend, pend_sc, facc[RT - 1][CT - 1]);
  }

  // Partial sums (constant share out) through LDS, one column tile at a time in two buffers; lane = token, registers
  // 4 g .. 4 g + 3 = outputs 8 g + 4 hf + 0..3.  Each thread then adds eight outputs of a token, in wavefront order.
  const float corr[2] = {__builtin_fmaf(W8_C0, csum[0], base[0]), __builtin_fmaf(W8_C0, csum[1], base[1])};
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    if (ct0 + c >= RTw) break;               // (uniform)
    const float out = second(c) ? corr[1] : corr[0];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v16f& f = facc[r][c];
        *(float4*)&part[c & 1][w][32 * r + l32][8 * g + 4 * hf] =
            make_float4(f[4 * g] - out, f[4 * g + 1] - out, f[4 * g + 2] - out, f[4 * g + 3] - out);
      }
    __syncthreads();
    const int n0 = (ct0 + c) * 32;
    for (int u = t; u < 32 * RT * 4; u += 64 * KS) {
      const int row = u >> 2, o = 8 * (u & 3), m = mt * 32 * RT + row;
      if (m >= M) continue;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = part[c & 1][0][row][o + e];
#pragma unroll
      for (int p = 1; p < KS; ++p)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += part[c & 1][p][row][o + e];
      if (bias) {
        const uint2 b0 = *(const uint2*)(bias + n0 + o), b1 = *(const uint2*)(bias + n0 + o + 4);
        v[0] += bf16_lo(b0.x); v[1] += bf16_hi(b0.x); v[2] += bf16_lo(b0.y); v[3] += bf16_hi(b0.y);
        v[4] += bf16_lo(b1.x); v[5] += bf16_hi(b1.x); v[6] += bf16_lo(b1.y); v[7] += bf16_hi(b1.y);
      }
      *(uint4*)(y + (size_t)m * N + n0 + o) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                        pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
  }
}

// ---------------------------------------------------------------------------
void launch_w8a8_quantize(const void* a, int R, int K, int RP, bool negate_odd, int8_t* codes, float* scales,
                          hipStream_t stream) {
  const unsigned grid = (unsigned)((RP / QB) * (K / QB));
  // Above 128 MiB of input the layer gains 1 to 2 % by reading past the caches (75600 x 5120 2.177 -> 2.147 ms,
  // 32760 x 8960 608 -> 591 us); below it loses as much (4096 x 5120 145.6 -> 148.3 us).
  const bool stream_in = (size_t)R * K * 2 > ((size_t)128 << 20);
#define SLA_QUANTIZE(STREAM) w8a8_quantize_kernel<STREAM><<<grid, 256, 0, stream>>>((const bf16_t*)a, R, K, RP, negate_odd ? 1 : 0, codes, scales)
  if (stream_in) SLA_QUANTIZE(true); else SLA_QUANTIZE(false);
#undef SLA_QUANTIZE
}

void launch_w8a8_unpack(const int8_t* frag, const float* s, int R, int K, int RP, bool negate_odd, int8_t* codes,
                        float* scales, hipStream_t stream) {
  w8a8_unpack_kernel<<<2048, 256, 0, stream>>>(frag, s, R, K, RP, negate_odd ? 1 : 0, codes, scales);
}

template <int RT, int CT, int KS>
static void launch_splitk(const int8_t* x8, const float* sx, int MP, const int8_t* w8, const float* sw, const void* bias,
                          void* y, int M, int N, int K, hipStream_t stream) {
  const int MT = (M + 32 * RT - 1) / (32 * RT), NT = N / (32 * CT);
  w8a8_gemm_splitk_kernel<RT, CT, KS><<<(unsigned)(8 * ((MT * NT + 7) / 8)), 64 * KS, 0, stream>>>(
      x8, sx, w8, sw, (const bf16_t*)bias, (bf16_t*)y, M, N, K, MP / 32, MP / QB, N / 32, N / QB, MT, NT);
}

template <int RT, int CT, int KS>
static void launch_wide(const int8_t* x8, const float* sx, int MP, const int8_t* w8, const float* sw, const void* bias,
                        void* y, int M, int N, int K, hipStream_t stream) {
  const int MT = (M + 32 * RT - 1) / (32 * RT), NT = (N / 32 + CT - 1) / CT;
  w8a8_gemm_wide_kernel<RT, CT, KS><<<(unsigned)(8 * ((MT * NT + 7) / 8)), 64 * KS, 0, stream>>>(
      x8, sx, w8, sw, (const bf16_t*)bias, (bf16_t*)y, M, N, K, MP / 32, MP / QB, N / 32, N / QB, MT, NT);
}

void launch_w8a8_gemm(const int8_t* x8, const float* sx, int MP, const int8_t* w8, const float* sw,
                      const void* bias, void* y, int M, int N, int K, hipStream_t stream) {
  const int MT = MP / W8_WG_M, NT = N / W8_WG_N, KB = K / QB;
  // Large tiles once they occupy most compute units, small split tiles below that; of a short contraction splitting has
  // less to win, so its line lies lower.  Whole layer in us, large / small, around each line:
  // one or two feature blocks (128 tiles): 128 -> 1024 at 4096 tokens (128 tiles) 11.7 / 11.6, -> 256 at 23243 (182) 11.7 /
  //   12.9, -> 5120 at 4096 (640) 16.8 / 21.2; 256 -> 4096 at 1024 (128) 11.8 / 11.6, -> 2560 at 2048 (160) 12.2 / 12.7,
  //   -> 5120 at 4096 (640) 19.6 / 24.2;
  // three to five (160): 640 -> 1024 at 4096 (128) 15.2 / 14.2, -> 2048 at 2304 (144) 15.2 / 14.5, -> 2176 at 2304 (153)
  //   15.8 / 14.7, -> 1024 at 5120 (160) 15.4 / 15.3, -> 4096 at 1280 (160) 14.7 / 15.3, -> 1152 at 6400 (225) 17.3 / 18.3;
  //   384 -> 1024 at 4096 (128) 13.1 / 12.5, -> 4096 at 1280 (160) 12.8 / 13.2;
  // more (200): 1536 -> 1536 at 4096 (192) 26.2 / 24.8, -> 5120 at 1280 (200) 23.2 / 24.4; 5120 -> 1536 at 4096 (192)
  //   60.2 / 56.4, -> 5120 at 1280 (200) 54.7 / 55.0, -> 5120 at 1536 (240) 56.1 / 62.6.
  // Long contractions that do not fill the chip with large tiles: of the wide tiles the smallest that deal out in one round (a
  // wavefront per SIMD).  The product in us, before / wide: 3072 -> 1024 at 1280 tokens
  // (320 tiles of 64 x 64, taken as 64 x 96) 9.6 / 8.5, at 1024 (256 tiles) 9.2 / 9.1, -> 3072 at 640 (480, 64 x 128) 12.4 / 10.1;
  // 5120 -> 5120 at 256 14.9 / 13.0, 512 (64 x 160) 21.5 / 18.0, 768 (64 x 128, two wavefronts) 29.0 / 26.2, 1024 (64 x 160, two)
  // 37.4 / 31.4; 5120 -> 13824 at 128 20.9 / 17.0, 384 (128 x 96, two) 48.9 / 37.4; 8960 -> 1536 at 2048 (128 x 96) 39.2 / 33.2, 4096
  // 77.6 / 64.3; 2048 -> 2048 at 1024 9.4 / 8.4, 2048 16.2 / 14.8.  On the other side: 240 tiles (8960 -> 1536 at 640) 18.5 / 20.7;
  // in two rounds 5120 -> 5120 at 1280 49.1 / 55.8; 12 blocks (1536 -> 8960 at 256) 10.4 / 10.7.
  // The round has to be filled: products of 32 x 32 x 128 against those that its wavefronts would go through at full tiles and
  // the longest run of blocks (odd numbers of blocks deal out unevenly), 65 % with four wavefronts a tile, 75 % with two (4096
  // -> 4096 at 700, 64 x 128 by two, 69 %: 26.9 / 27.9), and of few blocks two wavefronts have to get the same number or
  // nearly (2176 -> 2560 at 2000, 10 of 17 blocks in the longer run: 28.2 / 29.1).  Below 36 blocks, where a wavefront's start
  // and the sums' way through LDS are a third of its life, rows of 32 tokens that do not exist count as idle with four
  // wavefronts (2560 -> 8960 at 129, where of six such rows five exist, 8.8 / 9.9; 3584 -> 12416 at 83 12.4 / 13.2), the round
  // has to be filled to 61 % of what is left, to 64 by 64 x 128, to 75 by 128 x 96, and tiles above 64 x 128 by runs of nearly
  // one length (2176 -> 1280 at 2290, runs of 4, 4, 4 and 5 blocks, 11.2 / 13.2; 3200 -> 3200 at 860 15.3 / 16.3), unless the
  // small tiles would be eight wavefronts' in more than one round (4096 -> 8832 at 80: 0.64 of their time; in one round 4096
  // -> 5376 at 140 9.3 / 9.9).  Of 342 sizes drawn at random, most of them near these lines, the wide tiles were slower by
  // more than 3 % in 46 without this paragraph, in 4 with it.
  // Up to 64 tokens it is the stream of the weights that counts, and more wavefronts ask for it (2048 -> 16384 at 33: 12.7 / 13.3).
  if (M > 64 && KB >= 16) {
    const long long tiles64 = (long long)((M + 63) / 64) * (N / 64), work = 4 * tiles64 * KB;
    const long long exist = (long long)((M + 31) / 32) * (N / 32) * KB;
    const bool any = KB >= 36 || (KB >= 32 && tiles64 > 256 && (long long)((M + 31) / 32) * (N / 64) < 512);
    auto one_round = [&](int rt, int ct, int ks) {
      const long long tiles = (long long)((M + 32 * rt - 1) / (32 * rt)) * ((N / 32 + ct - 1) / ct);
      const int run = 2 * (((KB + 1) / 2 + ks - 1) / ks);
      const long long full = 1024ll * rt * ct * run;
      if (tiles * ks > 1024 || 20 * work < (ks == 4 ? 13 : 15) * full || (ks == 2 && KB < 24 && 10 * KB < 9 * ks * run)) return false;
      if (any) return true;
      if (ks == 4 && rt * ct > 8 && 5 * KB < 4 * ks * run) return false;
      return ks == 2 || 100 * exist >= (rt == 4 ? 75 : ct == 4 ? 64 : 61) * full;
    };
#define W8_WIDE(RT, CT, KS) if (one_round(RT, CT, KS)) return launch_wide<RT, CT, KS>(x8, sx, MP, w8, sw, bias, y, M, N, K, stream)
    W8_WIDE(2, 3, 4);
    W8_WIDE(2, 4, 4);
    W8_WIDE(2, 5, 4);
    W8_WIDE(4, 3, 4);
    W8_WIDE(2, 4, 2);
    W8_WIDE(2, 5, 2);
    W8_WIDE(4, 3, 2);
#undef W8_WIDE
  }
  if (MT * NT < (KB <= 2 ? 128 : KB <= 5 ? 160 : 200)) {
    // Of the small variants the one with the most work per wavefront that still brings at least 1024 wavefronts,
    // one per SIMD (the product of 5120 -> 5120 at 1 token 6.0 us, 64 8.5, 256 16.1, 512 23.8, 1024 46).
    auto waves = [&](int rt, int ct, int ks) { return (long long)((M + 32 * rt - 1) / (32 * rt)) * (N / (32 * ct)) * ks; };
#define W8_SPLITK(RT, CT, KS) launch_splitk<RT, CT, KS>(x8, sx, MP, w8, sw, bias, y, M, N, K, stream)
    if (waves(2, 2, 1) >= 1024) W8_SPLITK(2, 2, 1);
    else if (waves(2, 2, 2) >= 1024) W8_SPLITK(2, 2, 2);
    else if (waves(1, 2, 2) >= 1024) W8_SPLITK(1, 2, 2);
    else if (waves(1, 2, 4) >= 1024 && KB >= 32) W8_SPLITK(2, 2, 8);  // (as many wavefronts; long runs: 128 tokens of 13824 features 23.2 against 28.5)
    else if (waves(1, 2, 4) >= 1024) W8_SPLITK(1, 2, 4);
    else if (waves(1, 1, 4) >= 1024) W8_SPLITK(1, 1, 4);
    else W8_SPLITK(1, 1, 8);
#undef W8_SPLITK
    return;
  }
  const unsigned grid = (unsigned)(8 * (MT >= W8_DEAL_MT ? (MT + 7) / 8 * NT : (MT * NT + 7) / 8));
  w8a8_gemm_kernel<<<grid, 256, 0, stream>>>(x8, sx, w8, sw, (const bf16_t*)bias, (bf16_t*)y, M, N, K, MP / 32,
                                             MP / QB, N / 32, N / QB, MT, NT);
}

}  // namespace sla
