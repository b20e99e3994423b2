// sparse_fwd: the block-sparse low-bit softmax branch with the linear branch fused
// into its epilogue (Section 1.3: SLA computed by one low-bit attention kernel;
// Section 1.1: INT8 QK^T / FP8 PV in the SageAttention2++ manner).
//
// One workgroup per (b,h,query block); one wavefront per 32 queries.  Everything is
// computed transposed so that a lane owns ONE query (column) throughout:
//   S^T[key][query]  = K8 . Q8^T      v_mfma_i32_32x32x32_i8, A = K fragment (LDS), B = Q8 (registers)
//   P8 = e4m3(448 2^(t - r))          in registers; r = integer running reference of the query, shared
//                                     by its two lanes (lane, lane^32): one permlane swap per 32 keys
//   O^T[ch][query] += V8^T . P8^T     v_mfma_f32_32x32x64_f8f6f4, A = V fragment (LDS), B = P8 as it
//                                     sits in the accumulators' order (V was stored in that key order)
// so the rescale factor, the row sum and the final normalisation are per-lane scalars and P
// never touches LDS.  K/V fragments of the next critical blocks are copied global -> LDS
// asynchronously (no registers) into a ring of staging buffers while the current ones are
// consumed (one barrier per block).
//
// The kernel is bound by the vector ALU (exp2, FP8 packing, the row maximum), not by the matrix
// pipe, and a wavefront issues at most one vector instruction every ~5 cycles; so the main loop
// is arranged for every MFMA to have independent vector work of the same wavefront behind it:
// the two 32-key halves of a block are pipelined against each other (while the matrix pipe
// computes the scores of one half, the vector ALU turns the other half's scores into P codes),
// and the P.V product runs one block behind.  A query's reference level only ever rises and is
// usually final after a few blocks, so the step tests each half's maximum in its own lane first
// and joins the lane pairs, rounds up and rescales only when some lane of the wavefront passes.
//
// Epilogue: O_s = acc * delta_V / l;  optional linear term phi(Q) H_i / (phi(Q).Z_i) as bf16 MFMA
// (H_i already contains the output projection), bias, then a transposing pass through LDS so
// the global stores are row-contiguous.  Of a short list it is the longer part of a workgroup's life (7 key blocks: 13 000 of
// 36 000 cycles, 15 000 in the loop), a chain of waits for memory and of instructions: H_i is copied behind the list's last
// blocks, everything else requested in one go, softmax in phi(Q) left unnormalised, phi(Q).Z formed by the matrix pipe.
// Whole call: 24 slices of 4617 tokens 148.6 -> 143.3 us, 2 x 1024 30.7 -> 29.5, 12 x 32760 686 -> 677, 40 x 75600 9.42 -> 9.32 ms.
#include <type_traits>

#include "common.h"

namespace sla {

struct SparseDims {
  int N, Tq, Tk, n_c, total, per_xcd, phi, has_lin, out_f32, H;
  int q8_rows;       // rows per (b,h) of the Q code tensor (N rounded up to whole groups of 128)
  int TqW;           // workgroup tiles per (b,h)
  Layout lq, lo;  // of q and out
};
// The pointers are separate __restrict__ kernel parameters (not struct members) so the
// compiler knows the index list and the scales are never written by this kernel and can
// fetch them through the scalar unit.
struct SparseArgs {
  const bf16_t* __restrict__ q;
  const int8_t* __restrict__ q8;
  const int32_t* __restrict__ crit;
  const int8_t* __restrict__ k8;
  const uint8_t* __restrict__ v8;
  const float* __restrict__ dq;
  const float* __restrict__ dk;
  const float* __restrict__ dv;
  const bf16_t* __restrict__ HZ;
  const bf16_t* __restrict__ bias;
  void* __restrict__ out;
  float* __restrict__ lse;
  int N, Tq, Tk, n_c, total, per_xcd, phi, has_lin, out_f32, H;
  Layout lq, lo;
  int TqW, q8_rows;
};

constexpr int EPI_STRIDE = 32 * 4 + 16;         // bytes per staged output row (32 fp32 + pad)
// Score bias: the integer accumulators of the score MFMAs start from the bit pattern of the
// float 1/(2 pi), which the instruction takes as an inline constant (no registers).  A finished
// accumulator, reinterpreted as fp32, is then the float BIAS_F + s * 2^-26 exactly, for every
// score |s| <= 127 * 127 * 128 < 0x22F983 (the pattern stays inside the binade [1/8, 1/4)):
// no int -> float conversion is needed, and patterns order like the scores.
constexpr int BIAS_I = 0x3E22F983;
constexpr int BIAS_FLOOR = 0x3E000000;          // pattern below every reachable score (masked keys)
constexpr float SCORE_STEP = 1.0f / 67108864.f;  // 2^-26: what one score unit adds to the float

// Row state (per lane = per query): `r` is the running reference level, an INTEGER number of
// binary orders of magnitude (r = max over the 32-key tiles seen so far of ceil(log2(e) * row
// max)), so that P = 448 * 2^(t - r) <= 448 fits E4M3; `R` is the level the accumulators are
// expressed in.  Because r - R is an integer, a tile's contribution is brought to level R by
// the E8M0 block scale of the FP8 MFMA (2^(r-R) on the P operand): the accumulators are never
// rescaled on the vector ALU, except for a rare renormalisation when r - R exceeds 64.  The
// hardware takes the scale of a lane pair's registers 0..3 (keys 0..31 of the block) from the
// lower lane and that of registers 4..7 (keys 32..63) from the upper lane, so the two halves of
// a block may sit at different levels.  The row sum of the rounded P comes out of the same
// MFMA through a tile of ones.

__device__ __forceinline__ v4i as_v4i(const uint4& x) { return v4i{(int)x.x, (int)x.y, (int)x.z, (int)x.w}; }
__device__ __forceinline__ v8i as_v8i(const uint4& a, const uint4& b) {
  return v8i{(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
}

// Four consecutive 16-byte chunks (first, first + 1, ...) of a K or V record from LDS.
__device__ __forceinline__ void read4(const uint4* __restrict__ rec, int lane, int first, uint4 (&f)[4]) {
#pragma unroll
  for (int u = 0; u < 4; ++u) f[u] = rec[(first + u) * 64 + lane];
}

// One step (32 channels) of S^T = K8 . Q8^T for one 32-key half.
__device__ __forceinline__ v16i qk_step(const uint4& kf, const v4i& q8, const v16i& c) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(kf), q8, c, 0, 0, 0);
}

// One 32-channel tile of O^T += V8^T . P8^T, P scaled by 2^(scale_p - 127).
__device__ __forceinline__ void pv_tile(const uint4& v0, const uint4& v1, const v8i& pb, int scale_p, v16f& acc) {
  acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_v8i(v0, v1), pb, acc, 0, 0, 0, 127, 0, scale_p);
}
// The row sum of P through the ones tile, same scale.
__device__ __forceinline__ void pv_rowsum(const v8i& ones, const v8i& pb, int scale_p, v16f& accl) {
  accl = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ones, pb, accl, 0, 0, 0, 127, 0, scale_p);
}

// Maximum of this lane's 16 biased scores of one half (keys key0 .. key0 + 31), as a pattern.
template <bool tail>
__device__ __forceinline__ int half_max(v16i& s, int key0, int hf, int kvalid) {
  if (tail) {  // keys past the end of the sequence (last key block only) never win the max
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (key0 + 8 * (q >> 2) + 4 * hf + (q & 3) >= kvalid) s[q] = BIAS_FLOOR;
  }
  // two chains of three-operand maxima (7 + 9 values), joined at the end: 8 instructions
  int m0 = max(max(s[0], s[1]), s[2]), m1 = max(max(s[7], s[8]), s[9]);
  m0 = max(max(m0, s[3]), s[4]);
  m1 = max(max(m1, s[10]), s[11]);
  m0 = max(max(m0, s[5]), s[6]);
  m1 = max(max(m1, s[12]), s[13]);
  m1 = max(max(m1, s[14]), s[15]);
  return max(m0, m1);
}

// Per key block: the constants that turn a biased score pattern into exponents.  With
// c2s = c2 * 2^26 (c2 = log2(e) / sqrt(d) * delta_Q * delta_K) and x the pattern as a float,
//   t = c2 * s = fma(x, c2s, nb),   nb = -BIAS * c2s.
struct BlockConsts {
  float c2s;   // slope
  float nbg;   // nb + one score step: the guard keeps t - r <= 0 whatever the rounding of the products
  float lnb;   // log2(448) + nb: offs = lnb - r makes exp2(fma(x, c2s, offs)) = 448 * 2^(t - r)
};
__device__ __forceinline__ BlockConsts block_consts(float c2s) {
  // (explicit fused operations: the values must not depend on what the compiler chooses to contract)
  const float nb = -__int_as_float(BIAS_I) * c2s;
  return BlockConsts{c2s, __builtin_fmaf(c2s, SCORE_STEP, nb), __builtin_fmaf(c2s, -__int_as_float(BIAS_I), LOG2_448)};
}

// Row maximum over both lanes of the query -> new reference level r; returns offs (see above).
__device__ __forceinline__ float new_reference(int imax, const BlockConsts& bc, float pos_inf, float& r) {
  // after the swap one register holds the lower lane's value and the other the upper lane's, in both lanes
  const auto sw = __builtin_amdgcn_permlane32_swap(imax, imax, false, false);
  imax = max((int)sw[0], (int)sw[1]);
  const float cand = __builtin_ceilf(__builtin_fmaf(__int_as_float(imax), bc.c2s, bc.nbg));
  r = __builtin_amdgcn_fmed3f(r, cand, pos_inf);  // max(r, cand) in one instruction (both are finite)
  return bc.lnb - r;
}

// In-lane test value of a half's maximum: exceeds the (integer) reference level r exactly when the
// rounded-up level of this lane's scores would.
__device__ __forceinline__ float level_probe(int imax, const BlockConsts& bc) {
  return __builtin_fmaf(__int_as_float(imax), bc.c2s, bc.nbg);
}

// Four biased scores (accumulator registers 4g .. 4g+3 of one half) -> four FP8 codes of P in
// the returned word; `dst` supplies the register to overwrite half by half.
template <bool tail>
__device__ __forceinline__ int codes_quad(const v16i& s, int g, int key0, int hf, float c2s, float offs, int kvalid,
                                          int dst) {
  float p[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(__int_as_float(s[4 * g + e]), c2s, offs));
  if (tail) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (key0 + 8 * g + 4 * hf + e >= kvalid) p[e] = 0.f;
  }
  return cvt_pk_e4m3(p[2], p[3], cvt_pk_e4m3(p[0], p[1], dst, false), true);
}

// E8M0 code of 2^(r_prev - R): brings the P codes made at level r_prev to the accumulators'
// level R (r_prev - R <= 64 by the renormalisation rule; far below R the contribution vanishes).
// Rm127 = R - 127 is kept alongside R.
__device__ __forceinline__ int level_scale(float r_prev, float Rm127) {
  return (int)__builtin_amdgcn_fmed3f(r_prev - Rm127, 0.f, 254.f);
}

// Rare: the reference level has run more than 64 binades ahead of the accumulators' level
// (always so after the first block, whose R starts at "minus infinity"): bring them to level r.
__device__ __forceinline__ void renormalise(float r, float& R, float& Rm127, v16f (&acc)[4], v16f& accl) {
  const bool up = r - R > 64.f;
  const float down = up ? __builtin_amdgcn_exp2f(R - r) : 1.0f;
  if (up) {
    R = r;
    Rm127 = r - 127.f;
  }
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[ct][q] *= down;
#pragma unroll
  for (int q = 0; q < 16; ++q) accl[q] *= down;
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Workgroup barrier for the staging pipeline.  __syncthreads() would also wait for EVERY
// outstanding memory operation, including the asynchronous copies of the blocks still in
// flight, which is exactly what the pipeline must not do.  Each wavefront has already waited
// (s_waitcnt vmcnt) for its own pieces of the block being published and has consumed (through
// its MFMAs) every LDS read of the stage being retired, so a bare s_barrier is sufficient; the
// empty asm statements only stop the compiler from moving memory accesses across it.
__device__ __forceinline__ void stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Query blocks of 64 (NW = 2): a workgroup of two wavefronts per block, four of them on a compute unit.  Two
// wavefronts per SIMD need staging rings of at most 40 KiB, so K has three slots and V two (of 8 KiB each): K(b + 3)
// and V(b) are requested in step b, V at its start, and V has to land within the step -- the other three workgroups'
// arithmetic covers that.  (A workgroup of four wavefronts over the merged lists of two adjacent blocks fetched
// every record once for both, but a wavefront whose block did not have a key block idled through its step:
// 40 heads x 75600 tokens, top 15 %, whole call: 18.2 ms against 14.4 ms.)
// SHARED (query blocks of 64, NW = 4, every key block critical): all lists are the same, so a workgroup serves two
// adjacent query blocks, wavefronts 0-1 the first and 2-3 the second, and fetches every record once for both
// (12 heads x 32760 tokens, whole call: 3.43 ms against 3.90 ms one by one; 3.57 ms as merged lists).  Lists of 94 % of
// the blocks and more, but not all of them, are the one place where the merged lists were faster: 4 x 32760 tokens at
// 97 % 1.20 ms against 1.26 ms (at 90 % 1.27 against 1.23, at 75 % 1.18 against 1.06).
template <int NW, bool SHARED>
__global__ void __launch_bounds__(NW * 64, 2) sparse_fwd_kernel(
    const bf16_t* __restrict__ q_, const int8_t* __restrict__ q8_, const int32_t* __restrict__ crit_, const int8_t* __restrict__ k8_,
    const uint8_t* __restrict__ v8_, const float* __restrict__ dq_, const float* __restrict__ dk_,
    const float* __restrict__ dv_, const bf16_t* __restrict__ HZ_, const bf16_t* __restrict__ bias_,
    void* __restrict__ out_, float* __restrict__ lse_, const SparseDims dims) {
  static_assert(!SHARED || NW == 4, "shared lists: four wavefronts, two per query block of 64");
  const SparseArgs A = {q_, q8_, crit_, k8_, v8_, dq_, dk_, dv_, HZ_, bias_, out_, lse_, dims.N, dims.Tq, dims.Tk,
                        dims.n_c, dims.total, dims.per_xcd, dims.phi, dims.has_lin, dims.out_f32, dims.H,
                        dims.lq, dims.lo, dims.TqW, dims.q8_rows};
  constexpr int NT = NW * 64;
  constexpr int CH = 2 * (KV_FRAG_BYTES / 16) / NT;  // 16-byte chunks per thread per block
  constexpr int BQ = NW * 32;
  // Rings of four K and four V staging buffers, declared as separate objects so the compiler
  // can tell the asynchronous fill of one from the reads of another; after the main loop
  // the K slots hold H_i and wavefront w reuses V buffer w for the output transposition.
  __shared__ uint4 kst0[KV_FRAG_BYTES / 16], kst1[KV_FRAG_BYTES / 16], kst2[KV_FRAG_BYTES / 16], kst3[KV_FRAG_BYTES / 16];
  __shared__ uint4 vst0[KV_FRAG_BYTES / 16], vst1[KV_FRAG_BYTES / 16], vst2[KV_FRAG_BYTES / 16], vst3[KV_FRAG_BYTES / 16];
  constexpr int SLOT = KV_FRAG_BYTES / 16;
  __shared__ uint4 ring[5 * SLOT];
  constexpr bool SMALL = NW == 2;
  static_assert(32 * EPI_STRIDE <= KV_FRAG_BYTES, "output staging must fit one stage buffer");

  // Workgroup ids are dealt round-robin over the 8 XCDs.  All XCDs work on the SAME head at
  // the same time, each on its own contiguous eighth of that head's query blocks: the set of
  // K/V records in use chip-wide is then one head's (a few tens of MB, resident in the
  // Infinity Cache instead of being re-fetched from HBM), and the workgroups that share an
  // XCD's L2 are neighbouring query blocks, whose critical sets overlap.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  // (the division runs on the vector ALU; its uniform result goes back to scalar registers)
  const int bh = __builtin_amdgcn_readfirstlane(slot / A.per_xcd);  // per_xcd = ceil(TqW / 8)
  const int i = xcd * A.per_xcd + (slot - bh * A.per_xcd);       // workgroup tile (of BQ queries)
  if (i >= A.TqW) return;

  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l32 = lane & 31, hf = lane >> 5;
  // the query block whose scale and summaries this wavefront uses (an odd block count leaves the last
  // pair's second half without queries: clamped, nothing of it is stored)
  const int iq = SHARED ? min(2 * i + __builtin_amdgcn_readfirstlane(w >> 1), A.Tq - 1) : i;
  const int rowid = bh * A.Tq + iq;
  const int qrow = i * BQ + 32 * w + l32;
  const bool qok = qrow < A.N;
  const int b_ = __builtin_amdgcn_readfirstlane(bh / A.H), h_ = bh - b_ * A.H;
  const bf16_t* qptr = A.q + b_ * A.lq.sb + h_ * A.lq.sh + (qok ? qrow : 0) * A.lq.sn;

  // ---- Q block -> INT8 B operands (4 steps of 32 channels; this lane: 16 of each): the codes were made
  // with the block statistics (exact ties, see int8_code_word_exact); a lane half's 64 bytes are contiguous.
  const float dqi = A.dq[(size_t)rowid];
  v4i q8[4];
  {
    const v4i* src = (const v4i*)(A.q8 + ((size_t)bh * A.q8_rows + (qok ? qrow : 0)) * D + 64 * hf);
#pragma unroll
    for (int s = 0; s < 4; ++s) q8[s] = qok ? src[s] : v4i{0, 0, 0, 0};
  }
  const float cq = dqi * (LOG2E / 11.313708498984761f) * 67108864.f;  // log2(e) / sqrt(d) * delta_Q * 2^26 (see BIAS_I)

  v16f acc[4], accl = v16f{};
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = v16f{};
  // R starts far below any reachable level, so the first block renormalises (0 * 0) and sets R
  float r = -1e30f, R = -1e30f, Rm127 = -1e30f;
  float pos_inf = INFINITY;
  asm volatile("" : "+s"(pos_inf));  // in a scalar register: the third operand of the med3 that serves as max
  // A operand that sums P over the keys: FP8 1.0 in rows 0 and 4 of a 32-row tile, so the
  // row sum of a query lands in accumulator register 0 of both of its lanes.
  const int one4 = (l32 == 0 || l32 == 4) ? 0x38383838 : 0;
  v8i ones = {one4, one4, one4, one4, one4, one4, one4, one4};
  v16i bias16;
#pragma unroll
  for (int e = 0; e < 16; ++e) bias16[e] = BIAS_I;
  asm volatile("" : "+v"(bias16));  // kept in registers: the C operand of the first score MFMA of every half

  const int n_c = A.n_c;
  // the critical list and the K scales are read through the scalar unit (uniform addresses)
  const int32_t* __restrict__ crow = A.crit + ((size_t)bh * A.Tq + (SHARED ? 2 * i : i)) * n_c;
  const float* __restrict__ dkrow = A.dk + (size_t)bh * A.Tk;
  const size_t rec0 = (size_t)bh * A.Tk * KV_FRAG_BYTES;
  // Asynchronous global -> LDS copy of one block's K or V record (no registers in between).
  // Wavefront w copies the PW adjacent 1 KiB pieces [PW w, PW w + PW) of the record, lane l
  // supplying bytes [16 l, 16 l + 16) of a piece; the instruction's immediate offset is added
  // to the global and to the LDS address alike.
  constexpr int PW = CH / 2;
  static_assert(PW == 2 || PW == 4, "pieces per wavefront per record");
  const int w_s = __builtin_amdgcn_readfirstlane(w);  // wavefront index as a scalar
  const unsigned lane_off = (unsigned)(w * PW * 1024 + lane * 16);
  const char* const k8_bh = (const char*)A.k8 + rec0;  // this (b,h)'s records: uniform, loop invariant
  const char* const v8_bh = (const char*)A.v8 + rec0;
  // Written as inline assembly so that (a) the record's address stays in scalar registers (base +
  // j * 8 KiB by scalar arithmetic, one loop-invariant vector offset per lane) and (b) the compiler
  // does not know copies are in flight: it would otherwise make every LDS read it cannot prove
  // disjoint wait for ALL of them.  The pipeline waits for them by explicit counts (loads the
  // compiler does not know about only make its own waits more conservative).
  static_assert(KV_FRAG_BYTES == 1 << 13, "record size");
  auto copy_rec = [&](const char* rec, uint4* dst) {
    const unsigned lds_addr = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_ptr_t)(dst + w_s * PW * 64));
    if constexpr (PW == 2) {
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %1, %0\n\t"
                   "global_load_lds_dwordx4 %1, %0 offset:1024"
                   :
                   : "s"(rec), "v"(lane_off), "s"(lds_addr)
                   : "memory", "m0");
    } else {
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %1, %0\n\t"
                   "global_load_lds_dwordx4 %1, %0 offset:1024\n\t"
                   "global_load_lds_dwordx4 %1, %0 offset:2048\n\t"
                   "global_load_lds_dwordx4 %1, %0 offset:3072"
                   :
                   : "s"(rec), "v"(lane_off), "s"(lds_addr)
                   : "memory", "m0");
    }
  };
  auto fetch_rec = [&](const char* base_bh, int j, uint4* dst) { copy_rec(base_bh + (unsigned)__builtin_amdgcn_readfirstlane(j << 13), dst); };
  // K of list entry e; behind the list's end come the four quarters of H_i (one per output tile, as large as a record),
  // which the epilogue reads from the slots: copied in the last steps, where the copies past the end brought the last
  // block once more, they cost nothing, and the epilogue has no memory to wait for (it took them from memory tile by tile,
  // every wavefront for itself).
  const int k_end = A.has_lin ? n_c : 0x7fffffff;
  const char* const h_rec = (const char*)(A.HZ + (size_t)rowid * HZ_ELEMS);
  auto fetch_k = [&](int e, int j, uint4* dst) {
    copy_rec(e >= k_end ? h_rec + (unsigned)((e - k_end) << 13) : k8_bh + (unsigned)__builtin_amdgcn_readfirstlane(j << 13), dst);
  };
  auto fetch_k_in = [&](int, int j, uint4* dst) { fetch_rec(k8_bh, j, dst); };   // (an entry that the list has)
  auto dk_of = [&](int j) { return *(const float*)((const char*)dkrow + (unsigned)__builtin_amdgcn_readfirstlane(j << 2)); };
  const int kvalid_last = A.N - (A.Tk - 1) * BK;  // valid keys of the last key block
  const bool ragged = kvalid_last < BK;

  // Software pipeline over the critical list.  Entering step b, the scores of keys 0..31 of
  // block b (s0) are finished and the K fragments of its keys 32..63 (kfB) are in registers.
  // Step b has two phases of the same shape, each a chain of MFMAs with one piece of vector-ALU
  // work behind every MFMA (scheduling barriers pin the pieces there: a wavefront issues in
  // order, and the pieces execute while the MFMA in front of them runs):
  //   phase 1  MFMAs: scores of keys 32..63 of block b (s1), P.V tiles 0, 1 of block b-1
  //            vector: s0 -> maximum -> reference level -> FP8 codes of keys 0..31 of block b
  //   phase 2  MFMAs: scores of keys 0..31 of block b+1 (new s0), P.V tiles 2, 3 and the row sum
  //            of block b-1;  vector: s1 -> ... -> codes of keys 32..63 of block b
  // Each phase starts by reading from LDS the fragments the NEXT phase's MFMAs need (V of block
  // b-1, K of block b+1) and by starting the copy of K(b+4) resp. V(b+2) into the ring slot
  // retired in step b-1 (past the end of the list come the quarters of H_i in place of K, and V of the last block
  // again, into slots nothing reads any more: the step stays free of branches).  At its end the wavefront waits
  // for its own pieces of K(b+2) / V(b) and meets the others at one barrier, which publishes
  // those and retires K slot (b+1)%4 and V slot (b-1)%4.  The L2 / HBM latency of a block is thus
  // covered by the arithmetic of two to three steps.  A ragged last key block can only be the
  // last entry of the (ascending) list; it is peeled off the loop so that masking its missing
  // keys costs the other blocks nothing.
  const int last = n_c - 1;
  const bool has_tail = ragged && n_c > 0 && (crow[last]) == A.Tk - 1;
  // (SLA_FULL_WAITS: a checking build that waits for EVERY copy at each step instead of counting the
  // copies still allowed in flight; results must be bit-identical to the counting build.)
#ifdef SLA_FULL_WAITS
  constexpr int WAIT_KEEP2 = 0x0070;
#else
  constexpr int KEEP = SMALL ? PW : 2 * CH;           // copies that may stay in flight at the end of a step
  static_assert(KEEP < 16, "the low counter field");
  constexpr int WAIT_KEEP2 = 0x0070 | KEEP;           // s_waitcnt vmcnt(KEEP) lgkmcnt(0)
#endif
  constexpr int WAIT_ALL = 0x0070;                                            // s_waitcnt vmcnt(0) lgkmcnt(0)
  constexpr int WAIT_KEEP_ALL_VM = 0xC07F;                                    // s_waitcnt lgkmcnt(0) only (vmcnt 63)
  v16i s0, s1;
  v8i pb_a = {}, pb_b = {};   // P codes of blocks b-1 / b (alternating); all-zero codes contribute nothing
  uint4 kfA[4], kfB[4], vfa[4], vfb[4];
  int sc_prev = 127;          // E8M0 scale of the P codes of block b-1 (this lane's half of it)

#define SB __builtin_amdgcn_sched_barrier(0);
  // The reference bookkeeping is off the common path: a query's level r only ever rises, and after the first few blocks it has usually reached its
  // final value: a half's maximum is first tested in each lane alone (one fma and one compare: r
  // is an integer, so the rounded-up level of a lane pair exceeds r exactly when one of its two
  // lanes' own value does), and only if some lane of the wavefront passes does the wavefront join
  // the lane pairs, round up and raise r (a wave-uniform branch).  The exponent offset is formed
  // once per step, the scale of the codes just made is recomputed only in a step in which r moved
  // (and in the one after it, when the two halves of a block may still sit at different levels),
  // and the accumulators' level is looked at only then.
#define SLA_RAISE(IMAX)                                                                                \
  {                                                                                                   \
    const auto sw_ = __builtin_amdgcn_permlane32_swap(IMAX, IMAX, false, false);                      \
    const int im_ = max((int)sw_[0], (int)sw_[1]);                                                    \
    const float cand_ = __builtin_ceilf(__builtin_fmaf(__int_as_float(im_), bc_.c2s, bc_.nbg));       \
    r = __builtin_amdgcn_fmed3f(r, cand_, pos_inf);                                                   \
    offs_ = bc_.lnb - r;                                                                              \
    moved = 1;                                                                                        \
  }
#define SLA_STEP(B, FETCH_K, KNEXT, VPREV, KFILL, VFILL, PBP, PBN)                                  \
  {                                                                                                   \
    const int b_ = (B);                                                                               \
    /* ---- phase 1 */                                                                                \
    read4(VPREV, lane, 0, vfa);                                                                       \
    read4(KNEXT, lane, 0, kfA);                                                                       \
    if constexpr (SMALL) fetch_rec(v8_bh, j0, VFILL); else FETCH_K(b_ + 4, j4, KFILL);                \
    const int jn_ = crow[min(b_ + (SMALL ? 4 : 5), last)];                                            \
    const float dn_ = dk_of(SMALL ? j3 : j4);                                                         \
    const BlockConsts bc_ = block_consts(cq * d0);                                                    \
    float offs_ = bc_.lnb - r;                                                                        \
    const int moved_before = moved;                                                                   \
    moved = 0;                                                                                        \
    SB s1 = qk_step(kfB[0], q8[0], bias16);                                                           \
    SB const int mA_ = half_max<false>(s0, 0, hf, 0);                                                 \
    SB s1 = qk_step(kfB[1], q8[1], s1);                                                               \
    SB if (__any(level_probe(mA_, bc_) > r)) SLA_RAISE(mA_)                                           \
    const float rA_ = r;                                                                              \
    SB s1 = qk_step(kfB[2], q8[2], s1);                                                               \
    SB PBN[0] = codes_quad<false>(s0, 0, 0, hf, bc_.c2s, offs_, 0, PBN[0]);                           \
    SB s1 = qk_step(kfB[3], q8[3], s1);                                                               \
    SB PBN[1] = codes_quad<false>(s0, 1, 0, hf, bc_.c2s, offs_, 0, PBN[1]);                           \
    SB pv_tile(vfa[0], vfa[1], PBP, sc_prev, acc[0]);                                                 \
    SB PBN[2] = codes_quad<false>(s0, 2, 0, hf, bc_.c2s, offs_, 0, PBN[2]);                           \
    SB pv_tile(vfa[2], vfa[3], PBP, sc_prev, acc[1]);                                                 \
    SB PBN[3] = codes_quad<false>(s0, 3, 0, hf, bc_.c2s, offs_, 0, PBN[3]);                           \
    /* anchor: the branch below must not draw this phase's pieces past it */                          \
    asm volatile("" : "+v"(PBN), "+v"(s1), "+v"(acc[0]), "+v"(acc[1]));                               \
    /* ---- phase 2 */                                                                                \
    read4(VPREV, lane, 4, vfb);                                                                       \
    read4(KNEXT, lane, 4, kfB);                                                                       \
    if constexpr (SMALL) FETCH_K(b_ + 3, j3, KFILL); else fetch_rec(v8_bh, j2, VFILL);                \
    SB s0 = qk_step(kfA[0], q8[0], bias16);                                                           \
    SB const int mB_ = half_max<false>(s1, 32, hf, 0);                                                \
    SB s0 = qk_step(kfA[1], q8[1], s0);                                                               \
    SB if (__any(level_probe(mB_, bc_) > r)) SLA_RAISE(mB_)                                           \
    SB s0 = qk_step(kfA[2], q8[2], s0);                                                               \
    SB PBN[4] = codes_quad<false>(s1, 0, 32, hf, bc_.c2s, offs_, 0, PBN[4]);                          \
    SB s0 = qk_step(kfA[3], q8[3], s0);                                                               \
    SB PBN[5] = codes_quad<false>(s1, 1, 32, hf, bc_.c2s, offs_, 0, PBN[5]);                          \
    SB pv_tile(vfb[0], vfb[1], PBP, sc_prev, acc[2]);                                                 \
    SB PBN[6] = codes_quad<false>(s1, 2, 32, hf, bc_.c2s, offs_, 0, PBN[6]);                          \
    SB pv_tile(vfb[2], vfb[3], PBP, sc_prev, acc[3]);                                                 \
    SB PBN[7] = codes_quad<false>(s1, 3, 32, hf, bc_.c2s, offs_, 0, PBN[7]);                          \
    SB pv_rowsum(ones, PBP, sc_prev, accl);                                                           \
    if constexpr (SMALL) { j0 = j1; j1 = j2; j2 = j3; j3 = jn_; d0 = d1; d1 = d2; d2 = dn_; }         \
    else { j2 = j3; j3 = j4; j4 = jn_; d0 = d1; d1 = d2; d2 = d3; d3 = dn_; }                         \
    /* anchor: keeps every piece inside this step */                                                  \
    asm volatile("" : "+v"(PBN), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(accl),  \
                 "+v"(s0), "+s"(SMALL ? j3 : j4), "+s"(SMALL ? d2 : d3));                             \
    SB if (moved | moved_before) {                                                                    \
      if (__any(r - R > 64.f)) renormalise(r, R, Rm127, acc, accl);                                   \
      sc_prev = level_scale(hf ? r : rA_, Rm127);   /* level of this lane's half of the new codes */  \
    }                                                                                                 \
    __builtin_amdgcn_s_waitcnt(WAIT_KEEP2);                                                           \
    stage_barrier();                                                                                  \
  }
  auto k_slot = [&](int e) -> uint4* { const int x = e & 3; return x == 0 ? kst0 : x == 1 ? kst1 : x == 2 ? kst2 : kst3; };
  // What the epilogue needs of memory beside H_i, requested in one go behind the loop (one by one, each where it was used,
  // these loads were the longest part of a short list's workgroup): the wavefront's Q rows for phi(Q), two channels of
  // delta_V, Z_i and the bias per lane.
  uint4 qraw[8];
  float2 dv2 = make_float2(0.f, 0.f);
  uint32_t z2 = 0, b2 = 0;
  auto request_epilogue = [&]() __attribute__((always_inline)) {
    dv2 = *(const float2*)(A.dv + (size_t)bh * D + 2 * lane);
    if (!SHARED && A.has_lin) {
      const bf16_t* Hi = A.HZ + (size_t)rowid * HZ_ELEMS;
      z2 = *(const uint32_t*)(Hi + D * D + 2 * lane);
#pragma unroll
      for (int s = 0; s < 8; ++s)   // (rows beyond N come as row 0 of the slice; what they give is not stored)
        qraw[s] = *(const uint4*)(qptr + 32 * (s >> 1) + 16 * hf + 8 * (s & 1));
      if (A.bias) b2 = (uint32_t)A.bias[2 * lane] | (uint32_t)A.bias[2 * lane + 1] << 16;
    }
    asm volatile("" ::: "memory");   // (requested here, not where they are used)
  };
  int moved = 1;              // did the reference level of any query of this wavefront rise in the last step?

  if (n_c > 0) {  // (an empty list leaves only the linear term of the epilogue)
    // step 0 has no previous block: it multiplies all-zero P codes with this all-zero V slot
    uint4* const vzero = SMALL ? ring + 4 * SLOT : vst3;
    for (int e = t; e < KV_FRAG_BYTES / 16; e += NT) vzero[e] = make_uint4(0, 0, 0, 0);
    // indices of blocks 0..4 and K scales of blocks 0..3 (clamped to the list)
    int j0 = crow[0], j1 = crow[min(1, last)];
    int j2 = crow[min(2, last)], j3 = crow[min(3, last)], j4 = crow[min(4, last)];
    float d0 = dk_of(j0), d1 = dk_of(j1), d2 = dk_of(j2), d3 = dk_of(j3);
    // three groups of copies, in the order the steps will wait for them
    if constexpr (SMALL) {
      fetch_k(0, j0, ring);
      fetch_k(1, j1, ring + SLOT);
      fetch_k(2, j2, ring + 2 * SLOT);
    } else {
      fetch_k(0, j0, kst0);
      fetch_k(1, j1, kst1);
      fetch_k(2, j2, kst2);
      fetch_rec(v8_bh, j0, vst0);
      fetch_k(3, j3, kst3);
      fetch_rec(v8_bh, j1, vst1);
    }
    __builtin_amdgcn_s_waitcnt(WAIT_KEEP2);  // K(0), K(1) have landed
    stage_barrier();
    read4(SMALL ? ring : kst0, lane, 0, kfA);
    read4(SMALL ? ring : kst0, lane, 4, kfB);
    // Step 0 refills K slot 0 right away: every wavefront must have its fragments of block 0 in
    // registers before any wavefront starts that copy (inside the loop the barrier that ends a step
    // plays this part for the slot the next step refills).
    __builtin_amdgcn_s_waitcnt(WAIT_KEEP_ALL_VM);
    stage_barrier();
    s0 = qk_step(kfA[0], q8[0], bias16);
#pragma unroll
    for (int u = 1; u < 4; ++u) s0 = qk_step(kfA[u], q8[u], s0);
    const int nb_main = has_tail ? n_c - 1 : n_c;
    int b = 0;
    if constexpr (SMALL) {
      int kn = SLOT, k2 = 2 * SLOT, kf = 0;   // K slots of blocks b + 1, b + 2 and of the retired block b (filled with b + 3)
      uint4 *const v0 = ring + 3 * SLOT, *const v1 = ring + 4 * SLOT;
#define SLA_TURN { const int t_ = kn; kn = k2; k2 = kf; kf = t_; }
      for (; b + 2 <= nb_main; b += 2) {
        SLA_STEP(b, fetch_k, ring + kn, v1, ring + kf, v0, pb_b, pb_a)
        SLA_TURN
        SLA_STEP(b + 1, fetch_k, ring + kn, v0, ring + kf, v1, pb_a, pb_b)
        SLA_TURN
      }
      if (b < nb_main) {
        SLA_STEP(b, fetch_k, ring + kn, v1, ring + kf, v0, pb_b, pb_a)
        pb_b = pb_a;
      }
#undef SLA_TURN
      if (has_tail) {
        fetch_rec(v8_bh, j0, (last & 1) ? v1 : v0);               // (the main loop's steps copy their own block's V)
        if (A.has_lin) fetch_k(n_c + 2, 0, ring + last % 3 * SLOT);   // (and bring the first two quarters only)
      }
    } else {
      // (up to plain_end a step's K copy is of a block that the list has or, without a linear branch, of whatever: with the
      // choice in every step 12 x 32760 tokens, every block critical, took 0.5 % longer; query blocks of 64 do not care)
      const int plain_end = A.has_lin ? n_c - 4 : nb_main;
      for (; b + 4 <= plain_end; b += 4) {
        SLA_STEP(b, fetch_k_in, kst1, vst3, kst0, vst2, pb_b, pb_a)
        SLA_STEP(b + 1, fetch_k_in, kst2, vst0, kst1, vst3, pb_a, pb_b)
        SLA_STEP(b + 2, fetch_k_in, kst3, vst1, kst2, vst0, pb_b, pb_a)
        SLA_STEP(b + 3, fetch_k_in, kst0, vst2, kst3, vst1, pb_a, pb_b)
      }
      for (; b + 4 <= nb_main; b += 4) {
        SLA_STEP(b, fetch_k, kst1, vst3, kst0, vst2, pb_b, pb_a)
        SLA_STEP(b + 1, fetch_k, kst2, vst0, kst1, vst3, pb_a, pb_b)
        SLA_STEP(b + 2, fetch_k, kst3, vst1, kst2, vst0, pb_b, pb_a)
        SLA_STEP(b + 3, fetch_k, kst0, vst2, kst3, vst1, pb_a, pb_b)
      }
      // the (up to three) remaining steps keep the a/b alternation by copying the codes back
      if (b < nb_main) {
        SLA_STEP(b, fetch_k, kst1, vst3, kst0, vst2, pb_b, pb_a)
        pb_b = pb_a;
      }
      if (b + 1 < nb_main) {
        SLA_STEP(b + 1, fetch_k, kst2, vst0, kst1, vst3, pb_b, pb_a)
        pb_b = pb_a;
      }
      if (b + 2 < nb_main) {
        SLA_STEP(b + 2, fetch_k, kst3, vst1, kst2, vst0, pb_b, pb_a)
        pb_b = pb_a;
      }
    }
    if constexpr (!SMALL) {
      if (has_tail && A.has_lin) fetch_k(n_c + 3, 0, k_slot(n_c + 3));   // (the place of the last K block, which is consumed)
    }
    request_epilogue();
    if (has_tail) {  // the ragged last key block: s0 and kfB are ready, P.V of the block before it is due
      __builtin_amdgcn_s_waitcnt(WAIT_ALL);   // (its V is not waited for yet)
      stage_barrier();
      const int sp = (nb_main + 3) & 3;
      const uint4* vp = SMALL ? ring + (3 + (sp & 1)) * SLOT : sp == 0 ? vst0 : sp == 1 ? vst1 : sp == 2 ? vst2 : vst3;
      read4(vp, lane, 0, vfa);
      read4(vp, lane, 4, vfb);
      const BlockConsts bct = block_consts(cq * d0);
      s1 = qk_step(kfB[0], q8[0], bias16);
#pragma unroll
      for (int u = 1; u < 4; ++u) s1 = qk_step(kfB[u], q8[u], s1);
      pv_tile(vfa[0], vfa[1], pb_b, sc_prev, acc[0]);
      pv_tile(vfa[2], vfa[3], pb_b, sc_prev, acc[1]);
      pv_tile(vfb[0], vfb[1], pb_b, sc_prev, acc[2]);
      pv_tile(vfb[2], vfb[3], pb_b, sc_prev, acc[3]);
      pv_rowsum(ones, pb_b, sc_prev, accl);
      const int mAt = half_max<true>(s0, 0, hf, kvalid_last);
      const float offsAt = new_reference(mAt, bct, pos_inf, r);
      const float rAt = r;
      v8i pb_t = {};
#pragma unroll
      for (int g = 0; g < 4; ++g) pb_t[g] = codes_quad<true>(s0, g, 0, hf, bct.c2s, offsAt, kvalid_last, pb_t[g]);
      const int mBt = half_max<true>(s1, 32, hf, kvalid_last);
      const float offsBt = new_reference(mBt, bct, pos_inf, r);
#pragma unroll
      for (int g = 0; g < 4; ++g) pb_t[4 + g] = codes_quad<true>(s1, g, 32, hf, bct.c2s, offsBt, kvalid_last, pb_t[4 + g]);
      pb_b = pb_t;
      if (__any(r - R > 64.f)) renormalise(r, R, Rm127, acc, accl);
      sc_prev = level_scale(hf ? r : rAt, Rm127);
    }
    {  // P.V of the last block (it has landed: the last step, or the wait above, has waited for it)
      const int sl = last & 3;
      const uint4* vc = SMALL ? ring + (3 + (sl & 1)) * SLOT : sl == 0 ? vst0 : sl == 1 ? vst1 : sl == 2 ? vst2 : vst3;
      read4(vc, lane, 0, vfa);
      read4(vc, lane, 4, vfb);
      pv_tile(vfa[0], vfa[1], pb_b, sc_prev, acc[0]);
      pv_tile(vfa[2], vfa[3], pb_b, sc_prev, acc[1]);
      pv_tile(vfb[0], vfb[1], pb_b, sc_prev, acc[2]);
      pv_tile(vfb[2], vfb[3], pb_b, sc_prev, acc[3]);
      pv_rowsum(ones, pb_b, sc_prev, accl);
    }
  } else {
    if (A.has_lin) {
      if constexpr (SMALL) {
        for (int e = 0; e < 3; ++e) fetch_k(e, 0, ring + e * SLOT);
      } else {
        for (int e = 0; e < 4; ++e) fetch_k(e, 0, k_slot(e));
      }
    }
    request_epilogue();
  }
#undef SLA_STEP
#undef SLA_RAISE
#undef SB
  // Every copy has landed, H_i is published; nobody reads V any more: V slot w is wavefront w's own from here on (its LDS
  // operations execute in the order it issues them, only the compiler has to be kept from changing it).
  __builtin_amdgcn_s_waitcnt(WAIT_ALL);
  stage_barrier();
  uint4 h3[8];   // query blocks of 64, whose three K slots hold three quarters of H_i: the last one
  if (SMALL && A.has_lin) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) h3[ks] = *(const uint4*)(h_rec + (size_t)hz_frag_chunk(3, ks, lane) * 16);
  }
  unsigned char* my = (unsigned char*)(SMALL ? ring + (3 + w) * SLOT : w == 0 ? vst0 : w == 1 ? vst1 : w == 2 ? vst2 : vst3);
  // delta_V, Z_i and the bias, two channels of each per lane, laid out to be read by every lane
  *(float2*)(my + 8 * lane) = dv2;
  *(uint32_t*)(my + 512 + 4 * lane) = z2;
  *(uint32_t*)(my + 768 + 4 * lane) = b2;
  *(uint32_t*)(my + 1024 + 4 * lane) = 0u;
  __builtin_amdgcn_wave_barrier();

  // ---- normalise: O_s[q][ch] = acc * delta_V[ch] / l (+ the bias, which comes with the linear term only)
  const float ltot = accl[0];  // sum of the rounded P (scaled by 448), at level R
  const float inv_l = ltot > 0.f ? 1.0f / ltot : 0.f;
  if (A.lse && hf == 0 && qok)
    A.lse[(size_t)bh * A.N + qrow] = (R + __builtin_amdgcn_logf(ltot) - LOG2_448) * LN2;
  auto normalise = [&](auto bias) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = 32 * ct + 8 * g + 4 * hf;
        const float4 d4 = *(const float4*)(my + c * 4);
        const float dv4[4] = {d4.x, d4.y, d4.z, d4.w};
        uint2 b4 = make_uint2(0u, 0u);
        if (bias) b4 = *(const uint2*)(my + 768 + c * 2);
        const float bv[4] = {bf16_lo(b4.x), bf16_hi(b4.x), bf16_lo(b4.y), bf16_hi(b4.y)};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[ct][4 * g + e] = bias ? __builtin_fmaf(acc[ct][4 * g + e], dv4[e] * inv_l, bv[e]) : acc[ct][4 * g + e] * (dv4[e] * inv_l);
      }
  };
  if (!SHARED && A.bias) normalise(std::true_type{}); else normalise(std::false_type{});

  // ---- linear branch: O_l^T[o][q] = sum_c H[o][c] phi(Q)[q][c], divided by phi(Q).Z (which comes out of the matrix pipe
  // like the row sum of P: a fifth tile with Z in rows 0 and 4 gives it in register 0 of both lanes of a query)
  if (!SHARED && A.has_lin) {
    uint4 bq[8];
    phi_q_operands(qraw, A.phi, bq);
    const unsigned char* zrow = my + (l32 == 0 || l32 == 4 ? 512 : 1024) + 32 * hf;
    const uint4* h[4];
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) h[ot] = (SMALL ? ring + (n_c + ot) % 3 * SLOT : k_slot(n_c + ot)) + lane;
    auto h_op = [&](int ot, int ks) __attribute__((always_inline)) { return SMALL && ot == 3 ? h3[ks] : h[ot][ks * 64]; };
    v16f den = v16f{}, al[2] = {v16f{}, v16f{}};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      den = mfma_bf16(*(const uint4*)(zrow + 64 * (ks >> 1) + 16 * (ks & 1)), bq[ks], den);
      al[0] = mfma_bf16(h_op(0, ks), bq[ks], al[0]);
      al[1] = mfma_bf16(h_op(1, ks), bq[ks], al[1]);
    }
    const float inv_den = den[0] != 0.f ? 1.0f / den[0] : 0.f;  // no marginal block: no linear term
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[2 * half + u][r] = __builtin_fmaf(al[u][r], inv_den, acc[2 * half + u][r]);
      if (half == 0) {
        al[0] = al[1] = v16f{};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          al[0] = mfma_bf16(h_op(2, ks), bq[ks], al[0]);
          al[1] = mfma_bf16(h_op(3, ks), bq[ks], al[1]);
        }
      }
    }
  }

  // ---- transpose through LDS (per wavefront, in its own slot) and store
  __builtin_amdgcn_wave_barrier();
  const int row0 = i * BQ + 32 * w;
  const size_t out0 = (size_t)(b_ * A.lo.sb + h_ * A.lo.sh + row0 * A.lo.sn);
  if (!A.out_f32) {
    store_rows(my, acc, lane, (bf16_t*)A.out + out0, A.lo.sn, A.N - row0);
    return;
  }
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {     // 32 channels in fp32 at a time
    __builtin_amdgcn_wave_barrier();   // (compiler fence: the stores below stay behind the reads of the pass before)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v16f& a = acc[ct];
      *(float4*)(my + l32 * EPI_STRIDE + (8 * g + 4 * hf) * 4) = make_float4(a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int rr = it * 8 + (lane >> 3), c4 = lane & 7;
      const float4 val = *(const float4*)(my + rr * EPI_STRIDE + c4 * 16);
      if (row0 + rr < A.N) *(float4*)((float*)A.out + out0 + rr * A.lo.sn + 32 * ct + 4 * c4) = val;
    }
  }
}

void launch_sparse_fwd(const void* q, const int8_t* q8, const Problem& p, const int32_t* crit, int n_c, const int8_t* k8,
                       const uint8_t* v8, const float* dq, const float* dk, const float* dv,
                       const bf16_t* HZ, const bf16_t* proj_b, int phi_kind, bool has_linear,
                       void* out, bool out_f32, float* lse, bool all_critical, hipStream_t stream) {
  SparseDims dm;
  dm.N = p.N;
  dm.Tq = p.Tq;
  dm.Tk = p.Tk;
  dm.n_c = n_c;
  dm.total = p.BH * p.Tq;
  dm.phi = phi_kind;
  dm.has_lin = has_linear ? 1 : 0;
  dm.out_f32 = out_f32 ? 1 : 0;
  dm.H = p.H;
  dm.q8_rows = (p.N + 127) / 128 * 128;
  dm.lq = p.lq;
  dm.lo = p.lo;
  const bool shared = p.block_q == 64 && all_critical;
  dm.TqW = shared ? (p.Tq + 1) / 2 : p.Tq;
  dm.per_xcd = (dm.TqW + 7) / 8;  // workgroup tiles of one head per XCD
  const bf16_t* bias = has_linear ? proj_b : nullptr;
  const unsigned grid = (unsigned)(8 * dm.per_xcd * p.BH);
#define SLA_SPARSE(NW, SHARED) sparse_fwd_kernel<NW, SHARED><<<grid, NW * 64, 0, stream>>>( \
      (const bf16_t*)q, q8, crit, k8, v8, dq, dk, dv, HZ, bias, out, lse, dm)
  if (shared) SLA_SPARSE(4, true);
  else if (p.block_q == 128) SLA_SPARSE(4, false);
  else SLA_SPARSE(2, false);
#undef SLA_SPARSE
}

}  // namespace sla
