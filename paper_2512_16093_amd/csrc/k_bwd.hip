// Backward pass of SLA, sparse branch (the operator of the paper's finetuning stage, Section 1.2):
// the gradient of the unquantised block-sparse softmax attention
//     O^s[n] = sum_{t in critical blocks of n's query block} softmax_t(Q[n].K[t] / sqrt(d)) V[t]
// with respect to Q, K and V, in bf16 on the matrix cores with fp32 accumulation.
//
//   bwd_lse_delta_kernel  per query block: online-softmax pass over its critical key blocks ->
//                       lse (base-2 log-sum-exp of the scaled scores) and delta = dO . O^s per token.
//   bwd_dq_kernel       per query block, over its critical key blocks:
//                       P = exp2(S - lse), dS = P o (dO V^T - delta), dQ += dS K / sqrt(d).
//   bwd_dkv_kernel      per key block, over the query blocks that hold it as critical:
//                       dV += P^T dO, dK += dS^T Q / sqrt(d).
//
// All products are formed transposed where that saves a shuffle: a wavefront owns 32 tokens, one per
// lane (two lanes per token, each with half of the rows of an accumulator tile), so row statistics
// stay inside a lane pair, and an accumulator tile converted to bf16 is directly the B operand of
// the next product (its contraction index = the accumulator's rows).
//
// Operand tiles (32 tokens x 128 channels) are staged in LDS row-major as they are in memory.  A
// product that contracts over the channels reads its operand with one 16-byte read per step; a
// product that contracts over the tile's tokens reads the same tile with the transposing LDS read
// of gfx950 (ds_read_b64_tr_b16), so no transposed copy of any tensor is ever made.
#include <algorithm>
#include <cfloat>
#include <initializer_list>

#include "common.h"
#include "delta.h"

namespace sla {

constexpr float QK_LOG2 = LOG2E / 11.313708498984761f;   // log2(e) / sqrt(d)
constexpr float INV_SQRT_D = 1.0f / 11.313708498984761f;

// The same operand as n_op straight from memory (a workgroup's own rows, read once).
// (x: the (b,h) slice's first token; sn: elements from one token to the next)
__device__ __forceinline__ void own_rows(const bf16_t* x, long long sn, long long row, int N, int hf, uint4 (&f)[8]) {
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) f[ks] = row < N ? *(const uint4*)(x + row * sn + 16 * ks + 8 * hf) : uint4{0u, 0u, 0u, 0u};
}
// A tensor's layout as the kernel uses it: the caller's (ST) or, for the instances that serve contiguous
// [B,H,N,d] tensors only, compile-time strides (the row stride then folds into the address arithmetic).
template <bool ST>
__device__ __forceinline__ Layout lay(const Layout& L, int H, int N) {
  if constexpr (ST) return L;
  else return Layout{(long long)H * N * D, (long long)N * D, (long long)D};
}
#define SLA_BWD_LAYOUTS                                                                                         \
  const Layout L_q = lay<ST>(dm.lq, dm.H, dm.N), L_k = lay<ST>(dm.lk, dm.H, dm.N), L_v = lay<ST>(dm.lv, dm.H, dm.N), \
               L_d = lay<ST>(dm.ld, dm.H, dm.N), L_dq = lay<ST>(dm.ldq, dm.H, dm.N), L_dk = lay<ST>(dm.ldk, dm.H, dm.N), \
               L_dv = lay<ST>(dm.ldv, dm.H, dm.N), L_o = lay<ST>(dm.lo, dm.H, dm.N);                              \
  (void)L_q; (void)L_k; (void)L_v; (void)L_d; (void)L_dq; (void)L_dk; (void)L_dv; (void)L_o;
// First token of slice bh = b H + h of a tensor laid out by L.
__device__ __forceinline__ const bf16_t* slice_of(const bf16_t* x, const Layout& L, int bh, int H) {
  const int b = bh / H;
  return x + b * L.sb + (bh - b * H) * L.sh;
}
__device__ __forceinline__ bf16_t* slice_of(bf16_t* x, const Layout& L, int bh, int H) {
  const int b = bh / H;
  return x + b * L.sb + (bh - b * H) * L.sh;
}

// ROWS consecutive token rows of a [N, 128] tensor -> LDS tile(s), through registers (loaded one
// step ahead).  NT threads take part.
template <int NT, int ROWS>
struct RowStage {
  static constexpr int PER = ROWS * 16 / NT;
  uint4 pf[PER];
  // Rows beyond N come as row N - 1 and without a branch: the caller gives such rows a weight of exactly zero and
  // wants every call to issue the same loads (N > 0).
  __device__ __forceinline__ void load_clamped(const bf16_t* x, long long sn, int r0, int N, int t) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int c = u * NT + t;
      const uint4 got = *(const uint4*)(x + (long long)min(r0 + (c >> 4), N - 1) * sn + (c & 15) * 8);
      pf[u] = got;  // (through a named value: assigning the dereferenced pointer straight to the member left the arrays in scratch memory)
    }
  }
  __device__ __forceinline__ void store(unsigned char* lds, int t) const {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int c = u * NT + t;
      *(uint4*)(lds + (c >> 4) * TP + (c & 15) * 16) = pf[u];
    }
  }
};

struct BwdDims {
  int N, Tq, Tk, n_c, T32q, H;
  Layout lq, lk, lv, ld;      // of q, k, v and dout (dq, dk, dv: ldq, ldk, ldv; the forward's out: lo)
  Layout ldq, ldk, ldv, lo;
};

// Workgroup -> (block, head) for a 1-D grid of 8 * ceil(T / 8) * BH workgroups.  Consecutive workgroup
// ids go to the 8 XCDs in turn; this order gives each XCD a contiguous run of a head's blocks, so
// the workgroups resident on one XCD at a time work on neighbouring blocks.  Returns false for the padding.
__device__ __forceinline__ bool xcd_block(int T, int& block, int& bh, int number = blockIdx.x) {
  const int per_xcd = (T + 7) >> 3, xcd = number & 7, slot = number >> 3;
  bh = slot / per_xcd;
  block = xcd * per_xcd + (slot - bh * per_xcd);
  return block < T;
}

// ---- asynchronous copies of 32-row tiles (32 x 256 bytes) global -> LDS, without registers in between
//
// A tile is eight pieces of 1 KiB (four rows); a wavefront's copy instruction writes one piece, lane l its bytes
// [16 l, 16 l + 16).  The copy cannot pad rows, so a row's sixteen 16-byte chunks are stored permuted, chunk c of row r
// at position c ^ swz(r): the 16 lanes of a group that read the same chunk of 16 consecutive rows hit all banks once
// (n_op_swz), and so do the 32 lanes that read a 4-row x 64-byte patch (t_op_swz).  The compiler does not know these
// copies are in flight (it would wait for all of them before every LDS read): the callers wait by count.
constexpr int SWZ_TILE_B = 32 * 256;
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
__device__ __forceinline__ void copy_piece(const char* base, unsigned off, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" : : "s"(base), "v"(off), "s"(lds_addr) : "memory", "m0");
}
__device__ __forceinline__ void copy_piece(const char* addr, unsigned lds_addr) {  // (an address per lane)
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(addr), "s"(lds_addr) : "memory", "m0");
}
// Two consecutive pieces of a tile (FIRST and the next one), of no lane (mask 0) or all of them (-1; no wavefront here ever
// has a lane switched off).  The instruction's immediate offset moves both addresses, so lds_tile is that of the
// wavefront's first piece and base, off as TileCopy::base3 and off3 give them.
template <int FIRST>
__device__ __forceinline__ void copy_pieces_if(long long mask, const char* base, unsigned off0, unsigned off1, unsigned lds_tile) {
  asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 exec, %4\n\t"
               "global_load_lds_dwordx4 %1, %0 offset:%5\n\t"
               "global_load_lds_dwordx4 %2, %0 offset:%6\n\ts_mov_b64 exec, -1"
               : : "s"(base), "v"(off0), "v"(off1), "s"(lds_tile), "s"(mask), "n"(FIRST * 1024), "n"(FIRST * 1024 + 1024) : "memory", "m0");
}
// One tensor's copies by the WAVES wavefronts of a workgroup, 8 / WAVES pieces each.
template <int WAVES>
struct TileCopy {
  static constexpr int PPW = 8 / WAVES;
  const char* slice;   // the (b,h) slice's first token
  long long snb;       // bytes from one token to the next
  unsigned odd;        // 0: 16-byte aligned rows at a stride that the 32-bit offsets below reach
  unsigned off[4];     // this lane's byte offset in pieces i, i + 4 of its wavefront
  int w, lane;
  __device__ __forceinline__ void init(const bf16_t* x, long long sn, int w_, int lane_) {
    slice = (const char*)x;
    snb = 2 * sn;
    odd = ((unsigned)(uintptr_t)x & 15u) | (unsigned)(snb >> 26);
    w = w_;
    lane = lane_;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + (lane >> 4);
      off[i] = (unsigned)((4 * PPW * w + r) * snb) + (((lane & 15) ^ swz(4 * PPW * w + r)) << 4);
    }
  }
  // For copies of several pieces with immediate offsets: piece i reads base3 + off3(i) + 1024 i.
  __device__ __forceinline__ const char* base3(int row0) const { return slice + row0 * snb - 3072; }
  __device__ __forceinline__ unsigned off3(int i) const { return off[i] + (3072 - 1024 * i); }
  __device__ __forceinline__ unsigned dst(unsigned lds_tile) const { return __builtin_amdgcn_readfirstlane(lds_tile + w * PPW * 1024); }
  // Are rows row0 .. row0 + rows - 1 whole, and their copies of the plain kind?  (uniform)
  __device__ __forceinline__ bool plain(int row0, int rows, int N) const { return row0 + rows <= N && odd == 0; }
  // rows row0 .. row0 + 31; rows beyond N come as row N - 1 (their weight is zero) or, if asked for, as zeros
  template <bool ZEROS = false>
  __device__ __forceinline__ void tile(int row0, int N, unsigned lds_tile) const {
    if (__builtin_expect(plain(row0, 32, N), 1)) {
      const char* b = slice + row0 * snb;
#pragma unroll
      for (int i = 0; i < PPW; ++i) copy_piece(i < 4 ? b : b + 16 * snb, off[i & 3], dst(lds_tile) + i * 1024);
    } else {
      tile_any<ZEROS>(row0, N, lds_tile);
    }
  }
  template <bool ZEROS = false>
  __device__ __forceinline__ void tile_any(int row0, int N, unsigned lds_tile) const {
    int ln = lane;
    asm volatile("" : "+v"(ln));            // (nothing of this path is worth a register outside of it)
#pragma unroll 1
    for (int i = 0; i < PPW; ++i) {
      const int r = 4 * (PPW * w + i) + (ln >> 4);
      const char* src = slice + min(row0 + r, N - 1) * snb + (((ln & 15) ^ swz(r)) << 4);
      if (ZEROS && row0 + r >= N) {         // (fewer copies may be under way then than the caller counts: it waits for all of them)
        *(__attribute__((address_space(3))) v4i*)(uintptr_t)(dst(lds_tile) + i * 1024 + ln * 16) = v4i{};
      } else if ((odd & 15u) == 0) {
        copy_piece(src, dst(lds_tile) + i * 1024);
      } else {
        // A contiguous tensor may start at any element.  The asynchronous copies take whole 16-byte units only, an
        // ordinary load takes any address: through a register.  (It has arrived before the next one is requested, so
        // waiting by count errs on the safe side.)
        v4i got;
        __builtin_memcpy(&got, src, 16);
        *(__attribute__((address_space(3))) v4i*)(uintptr_t)(dst(lds_tile) + i * 1024 + ln * 16) = got;
      }
    }
  }
};
// n_op on such a tile: swz_lane_offset once per lane, the step's bits flipped in.
__device__ __forceinline__ int swz_lane_offset(int l32, int hf) { return l32 * 256 + ((hf ^ swz(l32)) << 4); }
__device__ __forceinline__ uint4 n_op_swz(const unsigned char* tile, int lane_off, int ks) {
  return *(const uint4*)(tile + (lane_off ^ (ks << 5)));
}
// t_op on such a tile (the same lane, row and channel assignment).
__device__ __forceinline__ int swz_tr_lane_offset(int lane) {
  const int hf = lane >> 5, row = 4 * hf + ((lane & 15) >> 2), chunk = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  return row * 256 + ((chunk ^ swz(row)) << 4) + 8 * (lane & 1);
}
__device__ __forceinline__ uint4 t_op_swz(const unsigned char* tile, int tr_off, int ct, int s) {
  union { v4s h[2]; uint4 v; } u;
  u.h[0] = read_tr(tile + 16 * s * 256 + (tr_off ^ (ct << 6)));
  u.h[1] = read_tr(tile + (16 * s + 8) * 256 + (tr_off ^ (ct << 6) ^ (2 << 4)));   // (eight rows on: swz flips bit 1)
  return u.v;
}
// 64 consecutive floats global -> LDS, one per lane.
__device__ __forceinline__ void copy_floats(const float* base, unsigned off, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, %0" : : "s"(base), "v"(off), "s"(lds_addr) : "memory", "m0");
}
// Waits for all but KEEP of this wavefront's copies and for its LDS reads, then meets the workgroup's other wavefronts.
template <int KEEP>
__device__ __forceinline__ void copies_barrier() {
  static_assert(KEEP < 64, "the counter's range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070 | (KEEP & 15) | ((KEEP >> 4) << 14));  // vmcnt(KEEP) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// lse2[bh][row], delta[bh][row] for every token row of every query block (rows beyond N: lse2 = +inf, delta = 0, so that
// their P is exactly 0 wherever they are used):  delta = dO . O^s = sum_t P_t (dO . V_t), so no output is formed: two
// products (S, dP), an exponential, an addition and one fma per score, all in fp32.
//
// A wavefront owns QT tiles of 32 queries; with two an operand read from LDS serves two matrix products (with 32
// queries each the reads alone asked for all the LDS delivers).  K and V tiles of 32 keys travel in a ring of two each,
// copied one and a half steps ahead, 32 KB per workgroup, two wavefronts per SIMD; the exponentials are issued between
// the products of V.  Bound by power: 1.56 to 1.60 GHz with the matrix pipe 60 % busy.  Before (O formed from P in bf16, 32
// queries per wavefront, copies through registers): 40 heads x 75600 tokens 13.4 -> 12.3 ms, 12 x 32760 with query
// blocks of 64 1.19 -> 0.92 ms.
template <int WAVES, int QT, bool ST>
__global__ void __launch_bounds__(WAVES * 64, 2) bwd_lse_delta_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                                   const bf16_t* __restrict__ v, const bf16_t* __restrict__ dout,
                                                                   const int32_t* __restrict__ crit, float* __restrict__ lse2,
                                                                   float* __restrict__ delta, BwdDims dm) {
  __shared__ __attribute__((aligned(16))) unsigned char ring[4 * SWZ_TILE_B];  // K, V of even tiles, K, V of odd ones
  int i, bh;
  if (!xcd_block(dm.Tq, i, bh)) return;
  SLA_BWD_LAYOUTS
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  const int lane_off = swz_lane_offset(l32, hf);
  const int row0 = 32 * QT * (i * WAVES + w);
  uint4 qf[QT][8], dof[QT][8];
#pragma unroll
  for (int x = 0; x < QT; ++x) {
    // (rows beyond N come as row N - 1; what they give is not stored)
    const long long row = min(row0 + 32 * x + l32, dm.N - 1);
    const bf16_t *qr = slice_of(q, L_q, bh, dm.H) + row * L_q.sn + 8 * hf, *dr = slice_of(dout, L_d, bh, dm.H) + row * L_d.sn + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      qf[x][ks] = *(const uint4*)(qr + 16 * ks);
      dof[x][ks] = *(const uint4*)(dr + 16 * ks);
    }
  }
  float m[QT], l[QT], dl[QT];
#pragma unroll
  for (int x = 0; x < QT; ++x) {
    m[x] = -INFINITY;
    l[x] = 0.f;
    dl[x] = 0.f;
  }
  if (dm.n_c > 0) {
    const int32_t* __restrict__ crow = crit + ((size_t)bh * dm.Tq + i) * dm.n_c;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)ring;
    TileCopy<WAVES> ck, cv;
    ck.init(slice_of(k, L_k, bh, dm.H), L_k.sn, w, lane);
    cv.init(slice_of(v, L_v, bh, dm.H), L_v.sn, w, lane);
    constexpr int PPW = TileCopy<WAVES>::PPW;
    // the products of a K or V tile with both query tiles' rows; between(x, ks): vector work to issue behind each of them
    auto products = [&](const unsigned char* tile, const uint4 (&b)[QT][8], v16f (&acc)[QT], auto between) __attribute__((always_inline)) {
      int off = lane_off;
      asm volatile("" : "+v"(off));            // (one register for the eight addresses instead of eight)
#pragma unroll
      for (int x = 0; x < QT; ++x) acc[x] = v16f{};
#pragma unroll
      for (int g = 0; g < 2; ++g) {            // (four operands at a time: the registers hold no more)
        uint4 a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a[ks] = n_op_swz(tile, off, 4 * g + ks);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int x = 0; x < QT; ++x) {
            acc[x] = mfma_bf16(a[ks], b[x][4 * g + ks], acc[x]);
            between(x, 4 * g + ks);
            __builtin_amdgcn_sched_barrier(0);
          }
      }
    };
    auto step = [&](int key0, int jn, int half) __attribute__((always_inline)) {   // jn: the next block's index
      const unsigned char* kt = ring + half * 2 * SWZ_TILE_B;
      const unsigned char* vt = kt + SWZ_TILE_B;
      v16f s[QT], dp[QT];
      products(kt, qf, s, [](int, int) {});
#pragma unroll
      for (int x = 0; x < QT; ++x) {
        if (key0 + 32 > dm.N) {                // (uniform) only the sequence's last key block can hold keys that do not exist
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (key0 + 8 * (r >> 2) + 4 * hf + (r & 3) >= dm.N) s[x][r] = -INFINITY;
        }
        float mx = s[x][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[x][r]);
        // The reference m moves only when a score exceeds it by more than 2^8: P then stays below 2^8, harmless in fp32.
        if (__any(mx * QK_LOG2 > m[x] + 8.0f)) {
          mx = fmaxf(mx, partner_f32(mx)) * QK_LOG2;
          const float m_new = mx > m[x] + 8.0f ? mx : m[x];
          const float alpha = __builtin_amdgcn_exp2f(m[x] - m_new);
          m[x] = m_new;
          l[x] *= alpha;
          dl[x] *= alpha;
        }
      }
      copies_barrier<2 * PPW>();               // V of this tile has landed; its K tile is consumed
      ck.tile(64 * jn + 32 * half, dm.N, lds0 + half * 2 * SWZ_TILE_B);
      products(vt, dof, dp, [&](int x, int ks) __attribute__((always_inline)) {   // two of the exponentials behind every product
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          s[x][2 * ks + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[x][2 * ks + e], QK_LOG2, -m[x]));
          l[x] += s[x][2 * ks + e];
        }
      });
#pragma unroll
      for (int x = 0; x < QT; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) dl[x] = __builtin_fmaf(s[x][r], dp[x][r], dl[x]);
      // (anchor: the exponentials stay in their step -- sunk into the next one they took its registers)
#pragma unroll
      for (int x = 0; x < QT; ++x) asm volatile("" : "+v"(l[x]), "+v"(dl[x]));
      __builtin_amdgcn_sched_barrier(0);
      copies_barrier<2 * PPW>();               // K of the next tile has landed; this V tile is consumed
      cv.tile(64 * jn + 32 * half, dm.N, lds0 + (half * 2 + 1) * SWZ_TILE_B);
    };
    int j = crow[0];
    __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0): the wavefront's own rows are in
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      ck.tile(64 * j + 32 * half, dm.N, lds0 + half * 2 * SWZ_TILE_B);
      cv.tile(64 * j + 32 * half, dm.N, lds0 + (half * 2 + 1) * SWZ_TILE_B);
    }
    copies_barrier<3 * PPW>();
    for (int b = 0; b < dm.n_c; ++b) {
      const int jn = crow[min(b + 1, dm.n_c - 1)];   // (after the last block: the last one again, into tiles nobody reads)
      step(64 * j, jn, 0);
      step(64 * j + 32, jn, 1);
      j = jn;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);        // (no copy may land after the workgroup has left)
  }
#pragma unroll
  for (int x = 0; x < QT; ++x) {
    const float lt = l[x] + partner_f32(l[x]), dt = dl[x] + partner_f32(dl[x]);
    const int row = row0 + 32 * x + l32;
    const bool live = row < dm.N && dm.n_c > 0;
    if (hf == 0) {
      const size_t idx = (size_t)bh * dm.T32q * 32 + row;
      lse2[idx] = live ? m[x] + __builtin_amdgcn_logf(lt) : INFINITY;
      delta[idx] = live ? dt / lt : 0.f;
    }
  }
}

// The unquantised SLA forward pass (Section 1.2's training-time operator), per query block over its critical key
// blocks with an online softmax: O = O^s + (phi(Q) H'_i) / (phi(Q) . Z_i) (+ b) in bf16, H'_i being the projected
// summaries the forward pass accumulates.
struct FwdEpilogue {
  const bf16_t* HZ;    // [BH, Tq, HZ_ROWS, D] or nullptr (no marginal block: no linear term)
  const bf16_t* bias;  // [D] or nullptr
  bf16_t* out;         // [BH, N, D]
  int phi;
  float* save_lse2;    // [BH, 32 T32q] or nullptr: the rows' log-sum-exp (base 2), as bwd_lse_delta_kernel writes it
  bf16_t* save_os;     // [BH, N, D] or nullptr: O^s alone (for delta = dO . O^s of a later backward pass)
  int* save_hdr;       // 64 words or nullptr: the saved state's header, zeros behind it (the first workgroup writes it)
  SavedHeader hdr;
  // CODES: q and k hold INT8 codes as bf16 numbers; a score is their (exact) product times
  // delta_Q[i] delta_K[j] / sqrt(d), and the feature map of the linear term reads the original Q
  const float* code_dq;  // [BH, Tq]
  const float* code_dk;  // [BH, Tk]
  const bf16_t* q_lin;   // the original Q, laid out by lq_lin
  Layout lq_lin;
};
//
// A wavefront owns 32 queries, K and V come in steps of KT tiles of 32 keys, copied one step ahead, and two wavefronts
// share a SIMD: one's exponentials hide behind the other's products and, 16 keys on, behind its own.  With four
// wavefronts two tiles a step (64 KB a workgroup, a barrier every 64 keys), with two one tile (32 KB: four workgroups
// stay on a compute unit; with two tiles there was one wavefront per SIMD, 12 x 32760 tokens 1280 instead of 1095 us a
// call; four wavefronts with one tile: 936 instead of 910).  Through registers (up to 64 of them) and with 78 KB for
// either size the call took: query blocks of 128, 12 x 32760 tokens 944 -> 863 us, 40 x 75600 15.1 -> 13.5 ms; of 64 1392 ->
// 1055 us, 23.0 -> 20.5 ms.  Bound, as counted at 40 x 75600: query blocks of 128 by power (1.58 GHz, the matrix pipe 65 %
// busy, 52 GB past L2 in 12.2 ms); of 64 by the stream of K and V, 32 KB for every 64 x 64 scores: 128 GB past L2 in 16.7 ms =
// 7.6 TB/s, what a plain reader of such tiles gets, with the pipe 44 % busy.  At 12 x 32760 the pipe is 57 and 50 % busy, 2.0
// and 4.4 GB go past L2 in 0.82 and 0.95 ms: the exponentials beside the products.
// The epilogue's H_i comes into the ring behind the loop (with two wavefronts half of it, the rest when the last step's tiles are
// consumed), its other operands in one go, phi(Q) is left unnormalised where that cancels, rows leave whole: attention kernel 750 ->
// 709 us at 12 x 32760 token-major with O^s saved; 4 x 2187, query blocks of 64 (19 us) no difference.  Asked for inside the last
// step, by a branch in the loop, H_i cost blocks of 64 with long lists more than it hid (whole call, in the loop / behind it /
// without any of this: 40 x 32760 at 10 % 3570 / 3415 / 3544, at 20 % 6411 / 5950 / 6134; 12 x 32760 1081 / 1070 / 1108; blocks of
// 128 at 30 % 6745 / 6705 / 6760).
template <int NW, bool CODES, bool ST>
__global__ void __launch_bounds__(NW * 64, 2) fwd_bf16_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                            const bf16_t* __restrict__ v, const int32_t* __restrict__ crit,
                                                            BwdDims dm, FwdEpilogue fe) {
  constexpr int KT = NW / 2, STEP_B = 2 * KT * SWZ_TILE_B;
  __shared__ __attribute__((aligned(16))) unsigned char ring[2 * STEP_B];  // two steps' tiles: KT of K, then KT of V
  __shared__ __attribute__((aligned(16))) unsigned char side[NW * 768];    // a wavefront's Z_i, bias, zeros
  int i, bh;
  if (fe.save_hdr && blockIdx.x == 0 && threadIdx.x < 64) {
    const int v[8] = {fe.hdr.magic, fe.hdr.B, fe.hdr.H, fe.hdr.N, fe.hdr.block_q, fe.hdr.n_c, fe.hdr.pad0, fe.hdr.pad1};
    int x = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if ((int)threadIdx.x == e) x = v[e];
    fe.save_hdr[threadIdx.x] = x;
  }
  if (!xcd_block(dm.Tq, i, bh)) return;
  SLA_BWD_LAYOUTS
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  const int T = i * NW + w;
  const long long qrow = 32ll * T + l32;
  const bool qok = qrow < dm.N;
  const size_t head = (size_t)bh * dm.N * D;   // (of the library's own contiguous tensors)
  const bf16_t* qh = slice_of(q, L_q, bh, dm.H);
  uint4 qf[8];
  own_rows(qh, L_q.sn, qrow, dm.N, hf, qf);
  const int32_t* __restrict__ crow = crit + ((size_t)bh * dm.Tq + i) * dm.n_c;
  v16f o[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) o[ct] = v16f{};
  float m = -FLT_MAX;    // (finite: a tile may hold no valid key, and then its P have to be 0 and not NaN)
  const float qscale = CODES ? QK_LOG2 * fe.code_dq[(size_t)bh * dm.Tq + i] : QK_LOG2;
  v16f lacc = v16f{};  // register 0: the running sum of P over the keys (see the ones operand below)
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)ring;
  // The epilogue's H_i (four quarters of 8 KB, one per output tile): as many as fit come into half `half` of the ring,
  // copied by all wavefronts.
  constexpr int H_HALF = STEP_B / 8192;        // quarters there: 4 or 2
  const char* const h_rec = (const char*)(fe.HZ + ((size_t)bh * dm.Tq + i) * HZ_ELEMS);
  auto request_h = [&](int half, int first) __attribute__((always_inline)) {   // quarters first .. first + H_HALF - 1
    if (fe.HZ) {
#pragma unroll
      for (int u = 0; u < STEP_B / 1024 / NW; ++u)
        copy_piece(h_rec + first * 8192, (unsigned)(1024 * (w + u * NW) + 16 * lane), lds0 + half * STEP_B + 1024 * (w + u * NW));
    }
  };
  if (dm.n_c > 0) {
    TileCopy<NW> ck, cv;
    ck.init(slice_of(k, L_k, bh, dm.H), L_k.sn, w, lane);
    cv.init(slice_of(v, L_v, bh, dm.H), L_v.sn, w, lane);
    const int n_off = swz_lane_offset(l32, hf), t_off = swz_tr_lane_offset(lane);
    auto request = [&](int key0, int half) __attribute__((always_inline)) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        ck.tile(key0 + 32 * kt, dm.N, lds0 + half * STEP_B + kt * SWZ_TILE_B);
        cv.template tile<true>(key0 + 32 * kt, dm.N, lds0 + half * STEP_B + (KT + kt) * SWZ_TILE_B);   // (zero times an infinite V would not be zero)
      }
    };
    // KT tiles of 32 keys from key0 on, in half `half` of the ring; next: the step behind this one starts there (< 0: none)
    auto step = [&](int key0, float c2, int half, int next) __attribute__((always_inline)) {   // c2: score -> base-2 logit
      copies_barrier<0>();                     // this step's tiles have landed; those of the step before are consumed
      if (next >= 0) request(next, half ^ 1);
      // (a half of the ring is a multiple of the bits that the reads flip: added to the lane's offset)
      int no = n_off + half * STEP_B, to = t_off + half * STEP_B;
      asm volatile("" : "+v"(no), "+v"(to));
      v16f s[KT];
      float mx = -INFINITY;
      uint4 ak[8], tv[2][4];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) ak[ks] = n_op_swz(ring, no, ks);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        s[kt] = v16f{};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {       // behind a product: the read of the next tile's operand, at the end V's first ones
          s[kt] = mfma_bf16(ak[ks], qf[ks], s[kt]);
          if (kt + 1 < KT) ak[ks] = n_op_swz(ring + (kt + 1) * SWZ_TILE_B, no, ks);
          else if (ks >= 4) tv[0][ks - 4] = t_op_swz(ring + KT * SWZ_TILE_B, to, ks - 4, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        if (key0 + 32 * kt + 32 > dm.N) {      // (uniform) only the sequence's last key block can hold keys that do not exist
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (key0 + 32 * kt + 8 * (r >> 2) + 4 * hf + (r & 3) >= dm.N) s[kt][r] = -INFINITY;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
      }
      // The reference m moves only when the tiles' maximum exceeds it by more than 2^8: P then stays below 2^8 (harmless
      // in bf16 and fp32) and the accumulators are rescaled a few times per row instead of every step.
      if (__any(mx * c2 > m + 8.0f)) {
        mx = fmaxf(mx, partner_f32(mx)) * c2;
        const float m_new = mx > m + 8.0f ? mx : m;
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        lacc[0] *= alpha;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[ct][r] *= alpha;
      }
      auto weight = [&](int e) __attribute__((always_inline)) {   // P of element e % 16 of tile e / 16
        s[e >> 4][e & 15] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e >> 4][e & 15], c2, -m));
      };
      const uint4 ones = uint4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};  // bf16 1.0: sums P over the keys
#pragma unroll
      for (int e = 0; e < 8; ++e) weight(e);
#pragma unroll
      for (int g = 0; g < 2 * KT; ++g) {       // 16 keys; behind their products the next ones' exponentials and operand reads
        const uint4 pb = acc_operand(s[g >> 1], g & 1);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          o[ct] = mfma_bf16(tv[g & 1][ct], pb, o[ct]);
          if (g + 1 < 2 * KT) {
            tv[(g + 1) & 1][ct] = t_op_swz(ring + (KT + ((g + 1) >> 1)) * SWZ_TILE_B, to, ct, (g + 1) & 1);
            weight(8 * g + 8 + 2 * ct);
            weight(8 * g + 9 + 2 * ct);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        lacc = mfma_bf16(ones, pb, lacc);      // every row of this tile = the key sum of P (as rounded for the product above)
      }
    };
    auto scale_of = [&](int j) __attribute__((always_inline)) { return CODES ? qscale * fe.code_dk[(size_t)bh * dm.Tk + j] : QK_LOG2; };
    int j = crow[0];
    request(64 * j, 0);
    // Where the loop lies within the 64-byte lines of the instruction cache is worth up to 2 % (12 x 32760, in steps of 8
    // bytes: 1081 us here and 24 bytes on, 1086 to 1100 at four of the other six places): it does not depend on the code ahead.
    if constexpr (KT == 1) asm volatile(".p2align 6\n\t.rept 4\n\ts_nop 0\n\t.endr");
    for (int b = 0; b < dm.n_c; ++b) {
      const int jn = crow[min(b + 1, dm.n_c - 1)], next = b + 1 < dm.n_c ? 64 * jn : -1;
      const float c2 = scale_of(j);
      if constexpr (KT == 2) {
        step(64 * j, c2, b & 1, next);
      } else {
        step(64 * j, c2, 0, 64 * j + 32);
        step(64 * j + 32, c2, 1, next);
      }
      j = jn;
    }
  }
  const int last_half = NW == 4 ? (dm.n_c - 1) & 1 : 1;   // of the ring, which the last step has read
  request_h(last_half ^ 1, 0);                 // (the last step does not read that half, and everybody is past the one before)
  // What the epilogue needs of memory beside that, in one go: Q for phi(Q), two channels of Z_i and of the bias per lane.
  uint4 qraw[8];
  uint32_t z2 = 0, b2 = 0;
  if (fe.HZ) {
    // (rows beyond N come as row N - 1: what they give is not stored)
    const long long row = qok ? qrow : dm.N - 1;
    const bf16_t* ql = CODES ? slice_of(fe.q_lin, fe.lq_lin, bh, dm.H) + row * fe.lq_lin.sn : qh + row * L_q.sn;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qraw[ks] = *(const uint4*)(ql + 32 * (ks >> 1) + 16 * hf + 8 * (ks & 1));
    z2 = *(const uint32_t*)(h_rec + D * D * 2 + 4 * lane);
    if (fe.bias) b2 = (uint32_t)fe.bias[2 * lane] | (uint32_t)fe.bias[2 * lane + 1] << 16;
  }
  if constexpr (H_HALF < 4) {                  // the other two quarters take the place of the last step's tiles
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    request_h(last_half, H_HALF);
  }
  const float l = lacc[0];
  const float inv_l = dm.n_c > 0 ? 1.0f / l : 0.f;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ct][r] *= inv_l;
  // what a backward pass needs of this one: the log-sum-exp, and O^s below
  if (fe.save_lse2 && hf == 0) fe.save_lse2[(size_t)bh * dm.T32q * 32 + 32 * T + l32] = (qok && dm.n_c > 0) ? m + __builtin_amdgcn_logf(l) : INFINITY;
  uint4 bq[8];
  if (fe.HZ) phi_q_operands(qraw, fe.phi, bq);
  copies_barrier<0>();                         // H_i has landed; nobody reads the last step's tiles any more
  const int rows = dm.N - 32 * T;              // of this wavefront's 32 that exist (32 and more: all)
  unsigned char* out_lds = ring + last_half * STEP_B + w * 8192;
  uint2 os[16];
  auto store_os = [&]() __attribute__((always_inline)) { store_rows(out_lds, os, lane, fe.save_os + head + 32ll * T * D, D, rows); };
  if (fe.save_lse2) {
    pack_rows(o, os);
    if (H_HALF == 4) store_os();               // (with less there, that half is still in use)
  }
  if (fe.HZ) {
    // linear term, transposed like everything else: O_l^T[o][n] = sum_c H'[c][o] phi(Q)[n][c]; the
    // stored chunks of H' are this product's A operand, phi(Q) follows their channel order.  phi(Q) . Z comes out of the
    // matrix pipe as well: a fifth tile with Z in rows 0 and 4 gives it in register 0 of both lanes of a query.
    unsigned char* my = side + 768 * w;
    *(uint32_t*)(my + 4 * lane) = z2;
    *(uint32_t*)(my + 256 + 4 * lane) = b2;
    *(uint32_t*)(my + 512 + 4 * lane) = 0u;
    __builtin_amdgcn_wave_barrier();
    const unsigned char* zrow = my + (l32 == 0 || l32 == 4 ? 0 : 512) + 32 * hf;
    auto h_op = [&](int ot, int ks) __attribute__((always_inline)) {
      return *(const uint4*)(ring + (ot < H_HALF ? last_half ^ 1 : last_half) * STEP_B + (ot % H_HALF * 8 + ks) * 1024 + 16 * lane);
    };
    v16f den = v16f{};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) den = mfma_bf16(*(const uint4*)(zrow + 64 * (ks >> 1) + 16 * (ks & 1)), bq[ks], den);
    const float inv_den = den[0] != 0.f ? 1.0f / den[0] : 0.f;  // no marginal block: no linear term
#pragma unroll
    for (int op = 0; op < 4; op += 2) {        // (two output tiles at a time: their products do not wait for each other)
      v16f al[2] = {v16f{}, v16f{}};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          al[u] = mfma_bf16(h_op(op + u, ks), bq[ks], al[u]);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[op + u][r] = __builtin_fmaf(al[u][r], inv_den, o[op + u][r]);
    }
    if (fe.bias) {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint2 b4 = *(const uint2*)(my + 256 + (32 * ct + 8 * g + 4 * hf) * 2);
          o[ct][4 * g] += bf16_lo(b4.x);
          o[ct][4 * g + 1] += bf16_hi(b4.x);
          o[ct][4 * g + 2] += bf16_lo(b4.y);
          o[ct][4 * g + 3] += bf16_hi(b4.y);
        }
    }
  }
  if constexpr (H_HALF < 4) {
    copies_barrier<0>();                       // (the quarters of H_i there are consumed)
    if (fe.save_lse2) store_os();
  }
  store_rows(out_lds, o, lane, slice_of(fe.out, L_o, bh, dm.H) + 32ll * T * L_o.sn, L_o.sn, rows);
}

// 4 accumulated values of one 8-channel group -> bf16, plus the linear branch's share if given.
__device__ __forceinline__ void store_grad4(bf16_t* dst, const float* lin, float a0, float a1, float a2, float a3) {
  if (lin) {
    const float4 x = *(const float4*)lin;
    a0 += x.x; a1 += x.y; a2 += x.z; a3 += x.w;
  }
  *(uint2*)dst = uint2{pack_bf16x2(a0, a1), pack_bf16x2(a2, a3)};
}

// Products whose result the vector ALU works on, written so that they sit in ordinary registers (where a wavefront has
// 512, the compiler put them into accumulation registers beside the sums and copied every element back).  The hardware
// does not hold back a vector instruction that reads a product's result, or writes its registers, too early (12 wait
// states after a product of this size on gfx950), and the compiler does not see these products.  score_done() hands a
// result over and has to stand behind at least two further products: a product is issued only when the one before has
// left the pipe (8 states), so they put 16 states between.  score_wait() is the wait by itself, where no products
// follow; also of a result that nobody reads, whose registers are given to something else from there on.
__device__ __forceinline__ void score0(v16f& d, const uint4& a, const v4i& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(__builtin_bit_cast(v4i, a)), "a"(b));
}
__device__ __forceinline__ void score_from(v16f& d, const uint4& a, const v4i& b, const v16f& c) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(__builtin_bit_cast(v4i, a)), "a"(b), "v"(c));
}
__device__ __forceinline__ void score(v16f& d, const uint4& a, const v4i& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(__builtin_bit_cast(v4i, a)), "a"(b));
}
__device__ __forceinline__ void score_done(v16f& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void score_wait(v16f& x) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(x)); }

// dQ, per query block over its critical key blocks: dS = P o (dP - delta) with P = 2^(S - lse), dQ += dS K / sqrt(d).
//
// A wavefront owns QT tiles of 32 queries (two: an operand read from LDS serves two products; with 32 queries each,
// the reads of four wavefronts at full matrix rate ask for all the LDS delivers), K and V come in tiles of 32 keys
// through a ring of R, copied up to R - 1 steps ahead.  A lone wavefront per SIMD, so a step is written in the order of
// issue, one piece per product, and runs across two tiles: S of tile t + 1 with dS of tile t behind its products, dQ of
// tile t with exponentials of tile t + 1, dP of tile t + 1 with the rest of them.  Operands are read a section early,
// and the barrier that publishes a tile stands in the middle of a section, whose products cover the first reads of it.
// 40 heads x 75600 tokens 16.8 -> 16.1 ms (half the LDS traffic lets the clock rise from 1.70 to 1.88 GHz; the matrix pipe
// was 56 % busy), query blocks of 64 (12 x 32760) 1.42 -> 1.00 ms.  A tile's copies go between the products of two sections, a
// pair at a time (in one burst behind the barrier they held the wavefront up), and dP starts from minus delta (32 of 325
// instructions of a step less): 16.1 -> 15.2 ms, 1.00 -> 0.93 ms.  With another 10 instructions and two waits of a step
// taken out it is no faster: bound by power (1.75 to 1.80 GHz, the matrix pipe 61 % busy).
// dq_block: one workgroup's part, `unit` counting workgroups of a slice (PER of them serve a query block: 32 WAVES QT rows
// each), in `ring` of dq_lds(WAVES) bytes.
constexpr int dq_ring(int waves) { return waves == 1 ? 2 : 4; }   // (four workgroups of one wavefront have 40 KB of LDS each)
constexpr int dq_lds(int waves) { return dq_ring(waves) * 2 * SWZ_TILE_B; }
template <int WAVES, int QT, bool ST>
__device__ __forceinline__ void dq_block(const bf16_t* __restrict__ q, const bf16_t* __restrict__ dout, const bf16_t* __restrict__ k,
                                         const bf16_t* __restrict__ v, const int32_t* __restrict__ crit,
                                         const float* __restrict__ lse2, const float* __restrict__ delta,
                                         const float* __restrict__ dq_lin, bf16_t* __restrict__ dq, const BwdDims& dm,
                                         unsigned char* ring, int unit, int per, int bh) {
  constexpr int R = dq_ring(WAVES);
  const int i = per == 1 ? unit : unit / per;
  SLA_BWD_LAYOUTS
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hf = lane >> 5;
  const int row0 = 32 * QT * (unit * WAVES + w);
  v4i qf[QT][8], dof[QT][8];
  v16f acc[QT][4];
  float lse[QT], del[QT];
  v16f from[QT];   // dP starts from minus delta (no subtraction per element)
#pragma unroll
  for (int x = 0; x < QT; ++x)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) acc[x][ct] = v16f{};
  if (dm.n_c > 0) {
    const int32_t* __restrict__ crow = crit + ((size_t)bh * dm.Tq + i) * dm.n_c;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)ring;
    TileCopy<WAVES> ck, cv;
    ck.init(slice_of(k, L_k, bh, dm.H), L_k.sn, w, lane);
    cv.init(slice_of(v, L_v, bh, dm.H), L_v.sn, w, lane);
    constexpr int PER_TILE = 2 * TileCopy<WAVES>::PPW;
    const int n_off = swz_lane_offset(l32, hf), t_off = swz_tr_lane_offset(lane);
    const int tiles = 2 * dm.n_c;
    auto block_at = [&](int b) __attribute__((always_inline)) { return crow[min(b, dm.n_c - 1)]; };   // (past the end: the last block again)
    auto request = [&](int tile, int key) __attribute__((always_inline)) {
      const unsigned dst = lds0 + (tile & (R - 1)) * 2 * SWZ_TILE_B;
      ck.tile(key, dm.N, dst);
      cv.tile(key, dm.N, dst + SWZ_TILE_B);
    };
    // The request under way: tile + R into the place of the tile consumed last, in pairs of pieces, K's first.
    constexpr int PAIRS = TileCopy<WAVES>::PPW;
    const int odd = (int)(ck.odd | cv.odd), always = ~((odd | -odd) >> 31);
    const char *rk = ck.base3(0), *rv = cv.base3(0);
    unsigned to_k = 0;
    int rmask = 0;                             // -1: all its rows exist and are copied the plain way, 0: it was made at once
    unsigned ok[4], ov[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ok[u] = ck.off3(u);
      ov[u] = cv.off3(u);
    }
    auto begin_request = [&](int tile, int key_) __attribute__((always_inline)) {
      const int key = __builtin_amdgcn_readfirstlane(key_);
      const unsigned dst = lds0 + (tile & (R - 1)) * 2 * SWZ_TILE_B;
      const int mask = always & ~((dm.N - 32 - key) >> 31);   // (by integer arithmetic: as a truth value the compiler kept it in vector registers)
      rmask = mask;
      rk = ck.base3(key);
      rv = cv.base3(key);
      to_k = ck.dst(dst);
      if (__builtin_expect(mask == 0, 0)) {
        ck.tile_any(key, dm.N, dst);
        cv.tile_any(key, dm.N, dst + SWZ_TILE_B);
      }
      return mask;
    };
    auto request_pair = [&](long long mask, int x) __attribute__((always_inline)) {
      const int first = 2 * x % PAIRS;         // of its tensor's pieces; four on the offsets repeat, sixteen rows on
      const char* from = (2 * x < PAIRS ? rk : rv) + (first < 4 ? 0 : 16 * ck.snb + (2 * x < PAIRS ? 0 : 16 * (cv.snb - ck.snb)));
      const unsigned(&o)[4] = 2 * x < PAIRS ? ok : ov;
      const unsigned to = to_k + (2 * x < PAIRS ? 0 : SWZ_TILE_B) + (first < 4 ? 0 : 4096);
      if (first & 2) copy_pieces_if<2>(mask, from, o[2], o[3], to); else copy_pieces_if<0>(mask, from, o[0], o[1], to);
    };
    // (names the place of what lives through the loop)
    auto hold = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < QT; ++x) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) asm volatile("" : "+a"(acc[x][ct]));
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+a"(qf[x][ks]), "+a"(dof[x][ks]));
        asm volatile("" : "+v"(from[x]));
      }
    };
#pragma unroll
    for (int tile = 0; tile < R; ++tile) request(tile, 64 * block_at(tile >> 1) + 32 * (tile & 1));
#pragma unroll
    for (int x = 0; x < QT; ++x) {
      // (rows beyond N come as row N - 1: their lse is +inf, so their P and dS are zero)
      const long long row = min(row0 + 32 * x + l32, dm.N - 1);
      const bf16_t *qr = slice_of(q, L_q, bh, dm.H) + row * L_q.sn + 8 * hf, *dr = slice_of(dout, L_d, bh, dm.H) + row * L_d.sn + 8 * hf;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        qf[x][ks] = *(const v4i*)(qr + 16 * ks);
        dof[x][ks] = *(const v4i*)(dr + 16 * ks);
      }
      const size_t sidx = (size_t)bh * dm.T32q * 32 + row0 + 32 * x + l32;
      lse[x] = lse2[sidx];
      del[x] = delta[sidx];
    }
    copies_barrier<0>();                       // (the wavefront's own rows and the first R tiles)
    uint4 ak[8], av[8], tk[4][2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) ak[ks] = n_op_swz(ring, n_off, ks);
    v16f sa[QT], sb[QT], dp[QT];
#pragma unroll
    for (int x = 0; x < QT; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) from[x][r] = -del[x];
    // the sequence's last key block can only be the last entry of the ascending list: from tile `whole` on keys are missing
    const int whole = crow[dm.n_c - 1] * 64 + 64 <= dm.N ? tiles : tiles - 2;
#define FENCE __builtin_amdgcn_sched_barrier(0);
    auto weight = [&](v16f (&s)[QT], int e) __attribute__((always_inline)) {   // P: element e % 16 of query tile e / 16
      s[e >> 4][e & 15] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e >> 4][e & 15], QK_LOG2, -lse[e >> 4]));
    };
    auto dscore = [&](v16f (&s)[QT], int e) __attribute__((always_inline)) { s[e >> 4][e & 15] *= dp[e >> 4][e & 15]; };
    // Keys beyond N (the sequence's last key block only) came as key N - 1, so their P and dS are finite: their column
    // of K^T is cleared.
    auto clear_missing = [&](int key0) __attribute__((always_inline)) {
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int key = key0 + 16 * y + 8 * (j >> 1) + 4 * hf + 2 * (j & 1);
          const uint32_t keep = (key < dm.N ? 0xffffu : 0u) | (key + 1 < dm.N ? 0xffff0000u : 0u);
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) {
            uint32_t* word = (uint32_t*)&tk[ct][y];
            word[j] &= keep;
          }
        }
    };
    // dP of a tile (V operands in av); behind its products the second part of its exponentials and, once the tile is
    // consumed and the next one has landed, the reads of the next one's K
    constexpr int M = 8 * QT, E = 16 * QT;   // products of a section; elements per lane of the query tiles' P, dS
    constexpr int EARLY = PAIRS / 2;         // pairs of the request that go behind the products of dP, the rest behind those of S
    auto dp_products = [&](v16f (&s)[QT], int tile, int key_far) __attribute__((always_inline)) {   // key_far: of tile + R
      const unsigned char* next = ring + ((tile + 1) & (R - 1)) * 2 * SWZ_TILE_B;
      int mask_next = 0;
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int ks = m / QT, x = m % QT;
        if (ks == 0) score_from(dp[x], av[0], dof[x][0], from[x]); else score(dp[x], av[ks], dof[x][ks]);
#pragma unroll
        for (int e = M - 3 + m * (E - M + 3) / M; e < M - 3 + (m + 1) * (E - M + 3) / M; ++e) weight(s, e);
        if (m == M / 2 - 1) {
          FENCE
          copies_barrier<(R - 2) * PER_TILE>();    // the next tile has landed; this one is consumed
          mask_next = begin_request(tile + R, key_far);
        }
        if (m >= M / 2 && (m - M / 2) % (M / 2 / EARLY) == M / 2 / EARLY - 1) request_pair(mask_next, (m - M / 2) / (M / 2 / EARLY));
        if (m >= M / 2 && x == 0) {
          ak[2 * (ks - 4)] = n_op_swz(next, n_off, 2 * (ks - 4));
          ak[2 * (ks - 4) + 1] = n_op_swz(next, n_off, 2 * (ks - 4) + 1);
        }
        FENCE
      }
    };
    {  // the first tile's S, P and dP
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int ks = m / QT, x = m % QT;
        if (ks == 0) score0(sa[x], ak[0], qf[x][0]); else score(sa[x], ak[ks], qf[x][ks]);
        if (x == 0) av[ks] = n_op_swz(ring + SWZ_TILE_B, n_off, ks);
        FENCE
      }
#pragma unroll
      for (int x = 0; x < QT; ++x) score_wait(sa[x]);
#pragma unroll
      for (int e = 0; e < M - 3; ++e) weight(sa, e);
#pragma unroll
      for (int y = 0; y < 8; ++y) tk[y & 3][y >> 2] = t_op_swz(ring, t_off, y & 3, y >> 2);
      if (whole <= 0) clear_missing(64 * crow[0]);
      dp_products(sa, 0, 64 * block_at(R / 2));
    }
    // One step: dQ of tile t from its P (s), dP and K^T operands; S, P, dP and operands of tile t + 1 (after the
    // last tile: of a copy of the last block, whose results nobody uses; a step that leaves them out made the
    // allocator spill 330 registers).
    auto step = [&](int t, v16f (&s)[QT], v16f (&sn)[QT], int key_far) __attribute__((always_inline)) {
      const unsigned char* kt = ring + ((t + 1) & (R - 1)) * 2 * SWZ_TILE_B;
      uint4 ds[QT][2];
      // dS of t, element by element, packed to operands as eight are done
      constexpr int E1 = QT == 2 ? E - 6 : E;      // of them behind the products of S (from the fourth on: dP of t is done)
      auto dscores = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int e = from; e < to; ++e) {
          dscore(s, e);
          if ((e & 7) == 7) ds[e >> 4][(e >> 3) & 1] = acc_operand(s[e >> 4], (e >> 3) & 1);
        }
      };
      int mask_now;
      // (carried round the loop in a vector register: the builtin folds away.  The wait state is for the instruction that
      // may have written that register just before: the compiler puts it behind its own lane reads only)
      asm("s_nop 1\n\tv_readfirstlane_b32 %0, %1" : "=s"(mask_now) : "v"(rmask));
      // S of t + 1; behind its products dS of t, the rest of the request and the reads of V
      constexpr int GAP = R == 2 ? 2 : M / (PAIRS - EARLY);   // (two tiles only: what is requested here is waited for this step)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int ks = m / QT, x = m % QT;
        if (ks == 0) score0(sn[x], ak[0], qf[x][0]); else score(sn[x], ak[ks], qf[x][ks]);
        if (m == 3) {
#pragma unroll
          for (int z = 0; z < QT; ++z) score_done(dp[z]);
        }
        if (m >= 3) dscores((m - 3) * E1 / (M - 3), (m - 2) * E1 / (M - 3));
        if (x == 0) av[ks] = n_op_swz(kt + SWZ_TILE_B, n_off, ks);
        if (m % GAP == GAP - 1 && m / GAP < PAIRS - EARLY) request_pair(mask_now, EARLY + m / GAP);
        FENCE
      }
      // dQ of t; behind its products the last of dS, the first part of the exponentials of t + 1 and its K^T operands
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int x = m >> 3, y = m & 7;
        acc[x][y & 3] = mfma_bf16(tk[y & 3][y >> 2], ds[x][y >> 2], acc[x][y & 3]);
        if (QT == 2 && m < 3) dscores(E1 + 2 * m, E1 + 2 * m + 2);
        if (m == 3) {
#pragma unroll
          for (int z = 0; z < QT; ++z) score_done(sn[z]);
        }
        if (m >= 3) weight(sn, m - 3);
        if (x == QT - 1) tk[y & 3][y >> 2] = t_op_swz(kt, t_off, y & 3, y >> 2);
        FENCE
      }
      if (__builtin_expect(t + 1 >= whole, 0)) clear_missing(64 * block_at((t + 1) >> 1) + 32 * ((t + 1) & 1));
      dp_products(sn, t + 1, key_far);
      hold();
    };
#undef FENCE
    hold();
    // (list entries are loaded a round before they are needed: a scalar load's latency in every step cost a tenth of it)
    int j0 = block_at(R / 2), j1 = block_at(R / 2 + 1);
    for (int t = 0; t < tiles; t += 2) {
      const int j2 = block_at(t / 2 + R / 2 + 2);
      step(t, sa, sb, 64 * j0 + 32);
      step(t + 1, sb, sa, 64 * j1);
      j0 = j1;
      j1 = j2;
    }
    // (the last step's dP is not used, but it is still on its way to its registers)
#pragma unroll
    for (int x = 0; x < QT; ++x) score_wait(dp[x]);
    __builtin_amdgcn_s_waitcnt(0x0F70);        // (no copy may land after the workgroup has left)
  }
#pragma unroll
  for (int x = 0; x < QT; ++x) {
    const long long row = row0 + 32 * x + l32;
    if (row >= dm.N) continue;
    const float* lin = dq_lin ? dq_lin + ((size_t)bh * dm.N + row) * D : nullptr;   // (the library's own tensor)
    bf16_t* dqrow = slice_of(dq, L_dq, bh, dm.H) + row * L_dq.sn;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int ch = 32 * ct + 8 * g + 4 * hf;
        const v16f& a = acc[x][ct];
        store_grad4(dqrow + ch, lin ? lin + ch : nullptr, a[4 * g] * INV_SQRT_D, a[4 * g + 1] * INV_SQRT_D,
                    a[4 * g + 2] * INV_SQRT_D, a[4 * g + 3] * INV_SQRT_D);
      }
  }
}
template <int WAVES, int QT, bool ST>
__global__ void __launch_bounds__(WAVES * 64, 1) bwd_dq_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ dout,
                                                              const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                                              const int32_t* __restrict__ crit, const float* __restrict__ lse2,
                                                              const float* __restrict__ delta, const float* __restrict__ dq_lin,
                                                              bf16_t* __restrict__ dq, BwdDims dm) {
  __shared__ __attribute__((aligned(16))) unsigned char ring[dq_lds(WAVES)];  // K, V tile by tile
  int i, bh;
  if (!xcd_block(dm.Tq, i, bh)) return;
  dq_block<WAVES, QT, ST>(q, dout, k, v, crit, lse2, delta, dq_lin, dq, dm, ring, i, 1, bh);
}

// The linear branch's share of dK and dV for the 32 keys of a wavefront (Section 1.2's operator:
// h_j = phi(K_j)^T V_j, z_j = column sums of phi(K_j), phi = softmax over the channels), given
// G_j = the sum of dH_i over the query blocks that hold key block j as marginal, and the same sum
// of dZ_i, in the summaries' storage order (hz_frag_chunk):
//     d phi(K)^T[c][n] = sum_o G[c][o] V[n][o] + dZ[c]   ->  dK[n] = phi o (d phi - phi . d phi)
//     dV^T[o][n]       = sum_c G[c][o] phi(K)[n][c]
// Called by the 128 threads of a key block with everything already on its way to registers: kr, vr the token's rows, g the
// block's chunks 128 u + t of G_j, z entries 2 (t % 64), 2 (t % 64) + 1 of its dZ.  G_j is published row by row ([o][c], pitch TP), so that the one product
// reads it as it is and the other with the transposing read.  Both barriers are inside.  Results in the accumulator
// layout of the sparse-branch kernels (lane = key, registers = channels).  Bound by its own chain of instructions: 23 000
// cycles of every workgroup when G_j was fetched chunk by chunk and transposed by 2-byte writes, now 10 000 (4 x 2187; whole
// backward pass with the requests ahead of the list, below, and the rows stored through LDS: 24 heads x 8000, query blocks
// of 64 1146 -> 1077 us, 40 x 75600 56.5 -> 54.6 ms).
constexpr int G_CHUNKS = D * D / 8 / 128;
template <int PHI>
__device__ __forceinline__ void linear_kv_share(const v4i (&kr)[8], const v4i (&vr)[8], bool ok, const v4i (&g)[G_CHUNKS], uint32_t z,
                                                unsigned char* gl, float* gz, int t, int lane, v16f (&dk_share)[4], v16f (&dv_share)[4]) {
  const int l32 = lane & 31, hf = lane >> 5, tr_off = tr_lane_offset(lane);
#pragma unroll
  for (int u = 0; u < G_CHUNKS; ++u) {
    const int x = u * 128 + t, ln = x & 63, ks = (x >> 6) & 7, ot = x >> 9;
    *(v4i*)(gl + (32 * ot + (ln & 31)) * TP + (32 * (ks >> 1) + 16 * (ln >> 5) + 8 * (ks & 1)) * 2) = g[u];
  }
  if (t < 64) *(float2*)(gz + 2 * t) = float2{bf16_lo(z), bf16_hi(z)};
  // phi(K[n]) at channels 16 ks + 8 hf + kk
  float cv[64];
  uint4 cf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) unpack8(__builtin_bit_cast(uint4, kr[ks]), &cv[8 * ks]);
  float kmax = 0.f, sum = 1.0f;
  if constexpr (PHI == 0) {
    kmax = cv[0];
#pragma unroll
    for (int e = 1; e < 64; ++e) kmax = fmaxf(kmax, cv[e]);
    kmax = fmaxf(kmax, partner_f32(kmax));
    sum = 0.f;
#pragma unroll
    for (int e = 0; e < 64; ++e) {
      cv[e] = __builtin_amdgcn_exp2f((cv[e] - kmax) * LOG2E);
      sum += cv[e];
    }
    sum += partner_f32(sum);
  } else {
#pragma unroll
    for (int e = 0; e < 64; ++e) cv[e] = phi_value<PHI>(cv[e], 0.f, 1.0f);
  }
  const float rsum = ok ? 1.0f / sum : 0.f;  // keys beyond the sequence take no part
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) cv[8 * ks + kk] *= rsum;
    cf[ks] = pack8(&cv[8 * ks]);
  }
  __syncthreads();
#pragma unroll
  for (int ot = 0; ot < 4; ++ot) {   // (the operand reads of a tile grouped ahead of its products)
    uint4 a[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) a[ks] = n_op(gl + 32 * ot * TP, l32, hf, ks);
    __builtin_amdgcn_sched_barrier(0);
    dv_share[ot] = v16f{};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) dv_share[ot] = mfma_bf16(a[ks], cf[ks], dv_share[ot]);
  }
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) cf[ks] = pair_order(__builtin_bit_cast(uint4, vr[ks]));
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    uint4 a[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) a[ks] = t_op(gl + 32 * (ks >> 1) * TP, tr_off, ct, ks & 1);
    __builtin_amdgcn_sched_barrier(0);
    dk_share[ct] = v16f{};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) dk_share[ct] = mfma_bf16(a[ks], cf[ks], dk_share[ct]);  // d phi(K)^T for now
  }
  // through the feature map: phi at the accumulator's channels 32 ct + 8 g + 4 hf + e, from K again
  float sdot = 0.f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) cf[ks] = pair_order(__builtin_bit_cast(uint4, kr[ks]));
  auto k_at = [&](int ct, int g4, float (&xk)[4]) __attribute__((always_inline)) {
    const uint4& kk = cf[2 * ct + (g4 >> 1)];
    const uint32_t k0 = g4 & 1 ? kk.z : kk.x, k1 = g4 & 1 ? kk.w : kk.y;
    xk[0] = bf16_lo(k0); xk[1] = bf16_hi(k0); xk[2] = bf16_lo(k1); xk[3] = bf16_hi(k1);
  };
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const float4 z4 = *(const float4*)(gz + 32 * ct + 8 * g4 + 4 * hf);
      const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
      float xk[4];
      k_at(ct, g4, xk);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dk_share[ct][4 * g4 + e] += zz[e];
        if constexpr (PHI == 0) sdot += phi_value<0>(xk[e], kmax, rsum) * dk_share[ct][4 * g4 + e];
      }
    }
  sdot += partner_f32(sdot);
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      float xk[4];
      k_at(ct, g4, xk);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        dk_share[ct][4 * g4 + e] = phi_backward<PHI>(xk[e], phi_value<PHI>(xk[e], kmax, rsum), dk_share[ct][4 * g4 + e], sdot);
    }
  __syncthreads();  // the published G is consumed: the caller may reuse the LDS
}

// The order in which dK/dV's workgroups (KB = 1) are started.  Their lists differ in length by more than threefold, and in the
// order of the key blocks the last long ones ran on alone: of 12 heads x 512 key blocks the slots stood empty for a
// seventh of the launch, of 40 x 1182 for 3.5 %.  Longest first (in classes of four query blocks) leaves 1 %; the order
// costs two small launches.  Each XCD orders its own eighth: of every eight consecutive key blocks one, at a place
// that changes from group to group.
__device__ __forceinline__ int dkv_dealt(int g, int xcd) { return 8 * g + ((xcd - (g + (g >> 3) + (g >> 6))) & 7); }
// counts[bh * Tk + j] = query blocks that hold key block j of slice bh as critical; 64 key blocks x 16 rows per workgroup.
__global__ void __launch_bounds__(1024) dkv_counts_kernel(const int8_t* __restrict__ mask, int Tq, int Tk, int* __restrict__ counts) {
  __shared__ int part[16][64];
  const int runs = (Tk + 63) / 64, bh = blockIdx.x / runs, l = threadIdx.x & 63, rg = threadIdx.x >> 6;
  const int j = 64 * (blockIdx.x - bh * runs) + l;
  const int8_t* col = mask + (size_t)bh * Tq * Tk + min(j, Tk - 1);
  int n = 0;
#pragma unroll 8
  for (int i = rg; i < Tq; i += 16) n += col[(size_t)i * Tk] == 1 ? 1 : 0;
  part[rg][l] = n;
  __syncthreads();
  if (rg == 0 && j < Tk) {
#pragma unroll
    for (int r = 1; r < 16; ++r) n += part[r][l];
    counts[(size_t)bh * Tk + j] = n;
  }
}
// order[xcd * per + slot] = first + x (x = bh * Tk + j of the ordered heads), lists of more query blocks first (-1: no
// workgroup); one workgroup per XCD.
constexpr int DKV_CLASSES = 2048;
__global__ void __launch_bounds__(1024) dkv_order_kernel(const int* __restrict__ counts, int total, int per, int first,
                                                         int* __restrict__ order) {
  __shared__ int start[DKV_CLASSES];   // of each class, the longest lists' first
  __shared__ int wsum[16];
  const int t = threadIdx.x, xcd = blockIdx.x, lane = t & 63, w = t >> 6;
  auto place = [&](int g) {            // class of this XCD's key block of group g
    const int x = dkv_dealt(g, xcd);
    return DKV_CLASSES - 1 - (x < total ? min(DKV_CLASSES - 1, 1 + (counts[x] >> 2)) : 0);
  };
  for (int c = t; c < DKV_CLASSES; c += 1024) start[c] = 0;
  __syncthreads();
  for (int g = t; g < per; g += 1024) atomicAdd(&start[place(g)], 1);
  __syncthreads();
  // exclusive sums over the classes, two per thread
  const int a = start[2 * t], b = start[2 * t + 1];
  int sum = a + b;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(sum, o);
    if (lane >= o) sum += up;
  }
  if (lane == 63) wsum[w] = sum;
  __syncthreads();
  int before = sum - a - b;
  for (int x = 0; x < w; ++x) before += wsum[x];
  start[2 * t] = before;
  start[2 * t + 1] = before + a;
  __syncthreads();
  // (which of two equally long lists goes first is left to the atomics: the results do not depend on the order)
  for (int g = t; g < per; g += 1024) {
    const int x = dkv_dealt(g, xcd), slot = atomicAdd(&start[place(g)], 1);
    order[(size_t)xcd * per + slot] = x < total ? first + x : -1;
  }
}

// One workgroup of four wavefronts per PAIR of adjacent key blocks (2 J, 2 J + 1): wavefronts 0, 1
// own the two key tiles of the first block, wavefronts 2, 3 those of the second (one key per lane
// pair).  The workgroup walks over the query blocks that hold either block as critical (found from
// the two mask columns; two flag bits per entry), staging each query tile's Q and dO once for both;
// a wavefront whose block is not critical for the current query block sits the step out.
// (KB = 2, 64 query rows per step.)  With KB = 1 a workgroup of two wavefronts serves one key block
// over its own list, 64 query rows per step as well, and two workgroups share a compute unit: every
// staged tile then serves one key block only, but no wavefront ever sits out.  With KB = 1 rows are copied straight to
// LDS (no registers, no padding: see TileCopy), the scores are formed in ordinary registers and dK, dV, K, V held in the
// accumulation registers, so a step has no register copies between the two files (there were 77, and the copies through
// registers took 56 more): 40 heads x 75600 tokens 29.9 -> 25.9 ms, 12 x 32760 token-major 2.18 -> 1.78 ms.  Cycle stamps
// then showed 3450 cycles a step for 2048 of products: 650 in which the next step's copies went out one behind another,
// 350 at the barrier, and the wavefront's own issue (a lone one gets an instruction away every five cycles or so).  With
// the copies between the products, two to an m0, the barrier ahead of the step's last section, the next step's first
// operands read behind that section's products and dP started from delta (no subtraction): 2900 cycles at 40 x 75600,
// 430 instructions instead of 504; whole backward pass 59.6 -> 57.8 ms (same box), 4 x 2187 (training step) 185 -> 180 us.
// Counted at 40 x 75600: 159 GB fetched past L2 at 6.6 to 6.9 TB/s, where a plain reader gets 6.9 to 7.6, and 1.67 to 1.72 GHz
// with the matrix pipe 56 % busy: bound by both, the stream and power.
// dkv_block: the part of workgroup `number` of `count`, in `lds`.
template <int KB, int TILES, int PHI, bool ST>
__device__ __forceinline__ void dkv_block(const bf16_t* __restrict__ q, const bf16_t* __restrict__ dout,
                                          const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                          const int8_t* __restrict__ mask, const float* __restrict__ lse2,
                                          const float* __restrict__ delta, const bf16_t* __restrict__ G,
                                          bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int pair_shift,
                                          const int* __restrict__ order, int natural, const BwdDims& dm, unsigned char* lds,
                                          int number, int count) {
  constexpr int NT = 128 * KB, ROWS = 32 * TILES;  // threads; query rows per step
  // two buffers of: Q (TILES tiles) then dO (TILES tiles) of ROWS consecutive query rows; then their lse, delta
  constexpr int BUF_B = KB == 1 ? 4 * SWZ_TILE_B : 2 * TILES * TILE_B;
  float (*stat)[2][ROWS] = (float (*)[2][ROWS])(lds + 2 * BUF_B);
  unsigned short* qlist = (unsigned short*)(lds + 2 * BUF_B + 2 * 2 * ROWS * 4);  // [Tq]
  __shared__ int wcnt[8][4];
  int J, bh;
  if (KB == 1 && number >= natural) {
    const int x = order[(number & 7) * ((count - natural) >> 3) + ((number - natural) >> 3)];   // (natural: a multiple of 8)
    if (x < 0) return;
    bh = x / dm.Tk;
    J = x - bh * dm.Tk;
  } else if (!xcd_block((dm.Tk + KB - 1) / KB, J, bh, number)) {
    return;
  }
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l32 = lane & 31, hf = lane >> 5;
  const int tr_off = tr_lane_offset(lane);
  const int half = KB == 2 ? w >> 1 : 0;
  SLA_BWD_LAYOUTS
  const bf16_t* kh = slice_of(k, L_k, bh, dm.H);
  const bf16_t* vh = slice_of(v, L_v, bh, dm.H);
  const bf16_t* qh = slice_of(q, L_q, bh, dm.H);
  const bf16_t* doh = slice_of(dout, L_d, bh, dm.H);
  const long long key = 64ll * (KB * J + half) + 32 * (w & 1) + l32;
  const bool kok = key < dm.N;
  // Everything that is needed ahead of the loop is requested before anything is waited for: the mask column(s) of the
  // first SCAN * NT query blocks, the wavefront's own rows, the block's G (one after the other they cost every
  // workgroup 18 000 cycles of 430 000 at 40 heads x 75600 tokens).
  constexpr int SCAN = 8;
  const bool has2 = KB == 2 && 2 * J + 1 < dm.Tk;
  const int8_t* mcol = mask + (size_t)bh * dm.Tq * dm.Tk + KB * J;
  int fl[SCAN];
  auto load_flags = [&](int base) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < SCAN; ++u) {
      const int8_t* m = mcol + (size_t)min(base + u * NT + t, dm.Tq - 1) * dm.Tk;
      fl[u] = (m[0] & 0xff) | (KB == 2 ? (has2 ? m[1] & 0xff : 0) << 8 : 0);
    }
  };
  load_flags(0);
  // (rows beyond N come as row N - 1: a finite value in a column that is never stored)
  v4i kf[8], vf[8];
  {
    const long long row = kok ? key : dm.N - 1;
    const bf16_t *kr = kh + row * L_k.sn + 8 * hf, *vr = vh + row * L_v.sn + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      kf[ks] = *(const v4i*)(kr + 16 * ks);
      vf[ks] = *(const v4i*)(vr + 16 * ks);
    }
  }
  v4i g[G_CHUNKS];
  uint32_t gz2 = 0;                      // (a pair of dZ: a single one, widened here, would be waited for here)
#pragma unroll
  for (int u = 0; u < G_CHUNKS; ++u) g[u] = v4i{};
  if (G) {
    const int jb = min(KB * J + half, dm.Tk - 1);  // (the missing second block of an odd last pair: its keys do not exist)
    const bf16_t* rec = G + ((size_t)bh * dm.Tk + jb) * HZ_ELEMS;
#pragma unroll
    for (int u = 0; u < G_CHUNKS; ++u) {
      const v4i got = *(const v4i*)(rec + (size_t)(u * 128 + (t & 127)) * 8);
      g[u] = got;
    }
    gz2 = *(const uint32_t*)(rec + D * D + 2 * (t & 63));
  }
  // ---- the query blocks of the key block(s), ascending; bit 14 / 15 = first / second block has it
  int nq = 0;
  for (int base = 0; base < dm.Tq; base += SCAN * NT) {
    if (base) {
      __syncthreads();                   // (the counts of the round before have been read)
      load_flags(base);
    }
    unsigned long long bal[SCAN];
#pragma unroll
    for (int u = 0; u < SCAN; ++u) {
      const int i = base + u * NT + t;
      fl[u] = i < dm.Tq ? ((fl[u] & 0xff) == 1 ? 1 : 0) | ((fl[u] >> 8) == 1 ? 2 : 0) : 0;
      bal[u] = __ballot(fl[u] != 0);
      if (lane == 0) wcnt[u][w] = __popcll(bal[u]);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < SCAN; ++u) {
      if (base + u * NT < dm.Tq) {       // (uniform)
        int off = nq + __popcll(bal[u] & ((1ull << lane) - 1ull));
#pragma unroll
        for (int x = 0; x < NT / 64; ++x) {
          const int n = wcnt[u][x];
          if (x < w) off += n;
          nq += n;
        }
        if (fl[u]) qlist[off] = (unsigned short)((base + u * NT + t) | (fl[u] << 14));
      }
    }
  }
  __syncthreads();                       // (the list is complete)
  // KB = 1: with V negated and the rows' delta in its registers beforehand the product gives delta - dP (no subtraction per
  // element), so dK collects with the other sign.
  constexpr float DK_SIGN = KB == 1 ? -1.0f : 1.0f;
  // the accumulators start from the linear branch's share (G = nullptr: there is none); dK is scaled
  // by 1 / sqrt(d) at the end, so its share goes in multiplied by sqrt(d)
  v16f dkt[4], dvt[4];
  if (G) {
    // each key block's two wavefronts publish its G_j in their own part of the (still unused) staging buffers
    static_assert(KB * 128 * TP <= 2 * BUF_B && KB * 128 <= 2 * 2 * ROWS, "the published G and dZ fit");
    linear_kv_share<PHI>(kf, vf, kok, g, gz2, lds + half * 128 * TP, (float*)stat + half * 128, t & 127, lane, dkt, dvt);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) dkt[ct][r] *= DK_SIGN * 11.313708498984761f;
  } else {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      dkt[ct] = v16f{};
      dvt[ct] = v16f{};
    }
  }
  if constexpr (KB == 1) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int e = 0; e < 4; ++e) vf[ks][e] ^= (int)0x80008000u;
  }
  // Steps = (list entry, pair of tiles of its query block): 64 query rows at a time.  With KB = 2 they travel
  // memory -> registers -> LDS: while step s is computed from one LDS buffer, step s + 1 is moved from
  // registers to the other buffer and step s + 2 is on its way from memory; one barrier per step.  Within a step
  // the two tiles are independent, which lets the matrix products of one run under the exponentials of the other.
  const int steps = __builtin_amdgcn_readfirstlane(nq << pair_shift), pair_mask = (1 << pair_shift) - 1;
  RowStage<NT, ROWS> sq0, sd0, sq1, sd1;
  float ps0 = 0.f, ps1 = 0.f;
  auto rows_of = [&](int step) { return ROWS * (((qlist[step >> pair_shift] & 0x3fff) << pair_shift) + (step & pair_mask)); };
#define DKV_LOAD(SQ, SD, PS, STEP)                                                                   \
  {                                                                                                  \
    const int r_ = rows_of(min((STEP), steps - 1));                                                  \
    SQ.load_clamped(qh, L_q.sn, r_, dm.N, t);                                                      \
    SD.load_clamped(doh, L_d.sn, r_, dm.N, t);                                                     \
    PS = ((t & ROWS) ? delta : lse2)[(size_t)bh * dm.T32q * 32 + r_ + (t & (ROWS - 1))];             \
  }
#define DKV_STORE(SQ, SD, PS, BUF)                                                                   \
  {                                                                                                  \
    SQ.store(lds + (BUF) * BUF_B, t);                                                                \
    SD.store(lds + (BUF) * BUF_B + TILES * TILE_B, t);                                               \
    if (t < 2 * ROWS) stat[BUF][t / ROWS][t & (ROWS - 1)] = PS;                                      \
  }
  auto compute = [&](int step, int buf) __attribute__((always_inline)) {
    if (!((qlist[step >> pair_shift] >> (14 + half)) & 1)) return;  // (wave-uniform)
    const unsigned char* qt0 = lds + buf * BUF_B;
    const unsigned char* dt0 = qt0 + TILES * TILE_B;
    v16f s[TILES], dp[TILES], p[TILES];
    // Operand reads are grouped ahead of the matrix products that use them (the compiler would
    // otherwise issue each read right before its product and wait for it every time).
#pragma unroll
    for (int u = 0; u < TILES; ++u) {
      uint4 aq[8], ad[8];
      float4 ls[4], dl[4];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        aq[ks] = n_op(qt0 + u * TILE_B, l32, hf, ks);
        ad[ks] = n_op(dt0 + u * TILE_B, l32, hf, ks);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        ls[g] = *(const float4*)&stat[buf][0][32 * u + 8 * g + 4 * hf];
        dl[g] = *(const float4*)&stat[buf][1][32 * u + 8 * g + 4 * hf];
      }
      s[u] = v16f{};
      dp[u] = v16f{};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        s[u] = mfma_bf16(aq[ks], __builtin_bit_cast(uint4, kf[ks]), s[u]);
        dp[u] = mfma_bf16(ad[ks], __builtin_bit_cast(uint4, vf[ks]), dp[u]);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, 24, 0);  // 24 LDS reads (operands, then lse and delta)
      __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);  // then 16 matrix products
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float lsv[4] = {ls[g].x, ls[g].y, ls[g].z, ls[g].w}, dlv[4] = {dl[g].x, dl[g].y, dl[g].z, dl[g].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pe = __builtin_amdgcn_exp2f(s[u][4 * g + e] * QK_LOG2 - lsv[e]);  // (a key beyond N: a finite value in a column that is never stored)
          p[u][4 * g + e] = pe;
          s[u][4 * g + e] = pe * (dp[u][4 * g + e] - dlv[e]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < TILES; ++u) {
#pragma unroll
      for (int sx = 0; sx < 2; ++sx) {
        const uint4 pb = acc_operand(p[u], sx), dsb = acc_operand(s[u], sx);
        uint4 td[4], tq[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          td[ct] = t_op(dt0 + u * TILE_B, tr_off, ct, sx);
          tq[ct] = t_op(qt0 + u * TILE_B, tr_off, ct, sx);
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          dvt[ct] = mfma_bf16(td[ct], pb, dvt[ct]);
          dkt[ct] = mfma_bf16(tq[ct], dsb, dkt[ct]);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);  // 16 transposing LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);   // then 8 matrix products
      }
    }
  };
  // One step: load step S + 2 into the set that step S has left, compute S, publish S + 1.  Every
  // step issues the same loads and stores whatever the step number (past the end the last step is
  // loaded again and a stale set is published to the buffer nobody reads any more; rows beyond N
  // come as row N - 1, their lse = +inf makes their P and dS exactly 0): with nothing conditional
  // the compiler can count the loads in flight and waits for those of step S + 1 only -- with the
  // loads under "if (step < steps)" it waited for everything, the loads just issued included,
  // before every publish, and again in the middle of the first group of products.
#define DKV_STEP(S, AHEAD, BUF, SQL, SDL, PSL, SQN, SDN, PSN)  \
  if ((S) >= steps) break;                                     \
  DKV_LOAD(SQL, SDL, PSL, (S) + (AHEAD))                       \
  compute((S), BUF);                                           \
  DKV_STORE(SQN, SDN, PSN, 1 - (BUF))                          \
  __syncthreads();
  if constexpr (KB == 1) {
    // Copies straight to LDS, two buffers; 16 pieces and one row of lse or delta per wavefront and step (past the end the
    // last step is copied again).  A lone wavefront per SIMD has nobody to fill the matrix pipe while it does anything
    // else, so a step is written in the order of issue, one piece per product, each ended by a full scheduling
    // fence: the exponentials, dS and conversions of one tile behind the products of the other, the LDS reads of a section
    // one section early, behind products that have just consumed the operands whose registers they take over, and the
    // barrier that publishes the next step's rows and frees this one's ahead of the last section, which needs no more
    // of them: behind its products the next step's first operands are read and the first copies of the step after it
    // requested, one per product (all at once they held the wavefront up for 650 of 3500 cycles, the path from
    // memory takes 64 bytes a cycle).
    if (steps > 0) {
      const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
      const int ws = __builtin_amdgcn_readfirstlane(w);
      TileCopy<2> cq, cd;
      cq.init(qh, L_q.sn, ws, lane);
      cd.init(doh, L_d.sn, ws, lane);
      const float* srow = (ws ? delta : lse2) + (size_t)bh * dm.T32q * 32;
      auto row_at = [&](int step) __attribute__((always_inline)) { return rows_of(min(step, steps - 1)); };
      auto request_stats = [&](int r0, int buf) __attribute__((always_inline)) { copy_floats(srow + r0, lane * 4, lds0 + 2 * BUF_B + (buf * 2 + ws) * ROWS * 4); };
      auto request = [&](int r0, int buf) __attribute__((always_inline)) {
        const unsigned to = lds0 + buf * BUF_B;
        cq.tile(r0, dm.N, to);
        cq.tile(r0 + 32, dm.N, to + SWZ_TILE_B);
        cd.tile(r0, dm.N, to + 2 * SWZ_TILE_B);
        cd.tile(r0 + 32, dm.N, to + 3 * SWZ_TILE_B);
        request_stats(r0, buf);
      };
      // the request under way, two pieces at a time: tile x / 2 of Q 0, Q 1, dO 0, dO 1, its first or last two pieces
      const char *rq = cq.base3(0), *rd = cd.base3(0);
      const int odd = (int)(cq.odd | cd.odd), always = ~((odd | -odd) >> 31);
      int rmask = 0;                     // -1: all its rows exist and are copied the plain way, 0: it was made at once
      unsigned oq[4], od[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        oq[i] = cq.off3(i);
        od[i] = cd.off3(i);
      }
      auto request_pieces = [&](long long mask, int x, int buf) __attribute__((always_inline)) {
        const int tile = x >> 1;
        const char* from = tile < 2 ? rq + (tile & 1) * 32 * cq.snb : rd + (tile & 1) * 32 * cd.snb;
        const unsigned(&o)[4] = tile < 2 ? oq : od;
        const unsigned to = cq.dst(lds0 + buf * BUF_B + tile * SWZ_TILE_B);
        if (x & 1) copy_pieces_if<2>(mask, from, o[2], o[3], to); else copy_pieces_if<0>(mask, from, o[0], o[1], to);
      };
      // (names the place of what lives through the loop: the allocator parked operands beside it otherwise)
      auto hold = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) asm volatile("" : "+a"(dkt[ct]), "+a"(dvt[ct]));
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+a"(kf[ks]), "+a"(vf[ks]));
      };
      const int n_off = swz_lane_offset(l32, hf), t_off = swz_tr_lane_offset(lane);
      uint4 aq[8], ad[8];                // tile 0's score operands
      v16f dp0;                          // and its rows' delta, where its dP starts from
#define FENCE __builtin_amdgcn_sched_barrier(0);
      auto read_delta = [&](v16f& x, int buf, int u, int g) __attribute__((always_inline)) {
        const float4 d4 = *(const float4*)&stat[buf][1][32 * u + 8 * g + 4 * hf];
        x[4 * g] = d4.x; x[4 * g + 1] = d4.y; x[4 * g + 2] = d4.z; x[4 * g + 3] = d4.w;
      };
      auto do_step = [&](int step, int buf) __attribute__((always_inline)) {
        const unsigned char *qt0 = lds + buf * BUF_B, *dt0 = qt0 + 2 * SWZ_TILE_B;
        const unsigned char *qn = lds + (1 - buf) * BUF_B, *dn = qn + 2 * SWZ_TILE_B;
        v16f s[2], dp[2];
        float4 ls[4];
        uint4 bq[8], bd[8];              // tile 1's score operands
        uint4 td[4], tq[4], te[4], tr[4];  // transposed operands of the gradient products, two sets in turn
        v4i pb[2][2], sb[2][2];          // P and minus dS of both tiles as operands
        float pe = 0.f, se = 0.f;        // the even element of the pair under way
        auto read_lse = [&](int u, int g) __attribute__((always_inline)) { ls[g] = *(const float4*)&stat[buf][0][32 * u + 8 * g + 4 * hf]; };
        auto anchor = [&](int u, int half) __attribute__((always_inline)) {  // (P and dS stay in their section: the compiler sank them past branches)
          asm volatile("" : "+v"(pb[u][half]), "+v"(sb[u][half]));
        };
        auto weight = [&](int e) __attribute__((always_inline)) {  // P and dS: accumulator register e % 16 of tile e / 16
          const int u = e >> 4, r = e & 15;
          const float4 l4 = ls[r >> 2];
          const float lv = (r & 3) == 0 ? l4.x : (r & 3) == 1 ? l4.y : (r & 3) == 2 ? l4.z : l4.w;
          const float p1 = __builtin_amdgcn_exp2f(s[u][r] * QK_LOG2 - lv);  // (a key beyond N: a finite value in a column that is never stored)
          const float s1 = p1 * dp[u][r];    // (minus dS)
          if (r & 1) {
            pb[u][r >> 3][(r & 7) >> 1] = (int)pack_bf16x2(pe, p1);
            sb[u][r >> 3][(r & 7) >> 1] = (int)pack_bf16x2(se, s1);
          } else {
            pe = p1;
            se = s1;
          }
        };
        int ahead = row_at(step + 2), mask_now;
        // (carried round the loop in a vector register: the builtin folds away.  The wait state is for the instruction that
        // may have written that register just before: the compiler puts it behind its own lane reads only)
        asm("s_nop 1\n\tv_readfirstlane_b32 %0, %1" : "=s"(mask_now) : "v"(rmask));
        // tile 0's scores
        dp[0] = dp0;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          if (ks == 0) score0(s[0], aq[0], kf[0]); else score(s[0], aq[ks], kf[ks]);
          bq[ks] = n_op_swz(qt0 + SWZ_TILE_B, n_off, ks);
          if (ks < 7) request_pieces(mask_now, 1 + ks, 1 - buf);      // (the rest of what the step before has begun to request)
          FENCE
          score(dp[0], ad[ks], vf[ks]);
          bd[ks] = n_op_swz(dt0 + SWZ_TILE_B, n_off, ks);
          if (ks >= 4) read_lse(0, ks - 4); else read_delta(dp[1], buf, 1, ks);
          FENCE
        }
        // tile 1's scores; P and dS of tile 0 from the fourth product on (its own are done then)
#pragma unroll
        for (int m = 0; m < 16; ++m) {
          const int ks = m >> 1;
          if (m & 1) {
            score(dp[1], bd[ks], vf[ks]);
          } else {
            if (ks == 0) score0(s[1], bq[0], kf[0]); else score(s[1], bq[ks], kf[ks]);
          }
          if (m == 3) {
            score_done(s[0]);
            score_done(dp[0]);
          }
          if (m >= 3) weight(m - 3);           // 0 .. 12
          if ((m & 3) == 1) td[m >> 2] = t_op_swz(dt0, t_off, m >> 2, 0);
          if ((m & 3) == 3) tq[m >> 2] = t_op_swz(qt0, t_off, m >> 2, 0);
          if (m >= 13) read_lse(1, m - 13);
          FENCE
        }
        anchor(0, 0);
        const int rows_ahead = __builtin_amdgcn_readfirstlane(ahead);
        // (by integer arithmetic: as a truth value the compiler kept it in vector registers)
        const int mask_next = always & ~((dm.N - ROWS - rows_ahead) >> 31);
        rmask = mask_next;
        rq = cq.base3(rows_ahead);
        rd = cd.base3(rows_ahead);
        // tile 0's gradient products, first half
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const int ct = m >> 1;
          if (m & 1) dkt[ct] = mfma_bf16(tq[ct], __builtin_bit_cast(uint4, sb[0][0]), dkt[ct]); else dvt[ct] = mfma_bf16(td[ct], __builtin_bit_cast(uint4, pb[0][0]), dvt[ct]);
          if (m < 3) weight(13 + m);
          if (m == 2) read_lse(1, 3);
          if (m == 3) {
            score_done(s[1]);
            score_done(dp[1]);
          }
          if (m >= 3) weight(16 + m - 3);      // 16 .. 20
          if (m & 1) tr[ct] = t_op_swz(qt0, t_off, ct, 1); else te[ct] = t_op_swz(dt0, t_off, ct, 1);
          FENCE
        }
        anchor(0, 1);
        // second half
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const int ct = m >> 1;
          if (m & 1) dkt[ct] = mfma_bf16(tr[ct], __builtin_bit_cast(uint4, sb[0][1]), dkt[ct]); else dvt[ct] = mfma_bf16(te[ct], __builtin_bit_cast(uint4, pb[0][1]), dvt[ct]);
          if (m < 6) weight(21 + m);           // 21 .. 26
          if (m & 1) tq[ct] = t_op_swz(qt0 + SWZ_TILE_B, t_off, ct, 0); else td[ct] = t_op_swz(dt0 + SWZ_TILE_B, t_off, ct, 0);
          FENCE
        }
        anchor(1, 0);
        // tile 1's, first half
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const int ct = m >> 1;
          if (m & 1) dkt[ct] = mfma_bf16(tq[ct], __builtin_bit_cast(uint4, sb[1][0]), dkt[ct]); else dvt[ct] = mfma_bf16(td[ct], __builtin_bit_cast(uint4, pb[1][0]), dvt[ct]);
          if (m < 5) weight(27 + m);           // 27 .. 31
          if (m & 1) tr[ct] = t_op_swz(qt0 + SWZ_TILE_B, t_off, ct, 1); else te[ct] = t_op_swz(dt0 + SWZ_TILE_B, t_off, ct, 1);
          FENCE
        }
        anchor(1, 1);
        copies_barrier<0>();             // the next step's rows have landed; this step's are consumed
        if (__builtin_expect(mask_next == 0, 0)) {
#pragma unroll 1
          for (int u = 0; u < 2; ++u) {
            cq.tile_any(rows_ahead + 32 * u, dm.N, lds0 + buf * BUF_B + u * SWZ_TILE_B);
            cd.tile_any(rows_ahead + 32 * u, dm.N, lds0 + buf * BUF_B + (2 + u) * SWZ_TILE_B);
          }
        }
        // second half
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const int ct = m >> 1;
          if (m & 1) dkt[ct] = mfma_bf16(tr[ct], __builtin_bit_cast(uint4, sb[1][1]), dkt[ct]); else dvt[ct] = mfma_bf16(te[ct], __builtin_bit_cast(uint4, pb[1][1]), dvt[ct]);
          aq[m] = n_op_swz(qn, n_off, m);
          ad[m] = n_op_swz(dn, n_off, m);
          if (m < 4) read_delta(dp0, 1 - buf, 0, m);
          if (m == 4) request_stats(rows_ahead, buf);
          if (m == 6) request_pieces(mask_next, 0, buf);
          FENCE
        }
        hold();
      };
      const int r0 = __builtin_amdgcn_readfirstlane(row_at(0)), r1 = __builtin_amdgcn_readfirstlane(row_at(1));
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the workgroup's own K, V rows are in
      request(r0, 0);
      request(r1, 1);
      copies_barrier<0>();
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        aq[ks] = n_op_swz(lds, n_off, ks);
        ad[ks] = n_op_swz(lds + 2 * SWZ_TILE_B, n_off, ks);
        if (ks < 4) read_delta(dp0, 0, 0, ks);
      }
      FENCE
      hold();
      for (int step = 0; step < steps; step += 2) {  // (every exit test is uniform over the workgroup)
        do_step(step, 0);
        if (step + 1 >= steps) break;
        do_step(step + 1, 1);
      }
#undef FENCE
      __builtin_amdgcn_s_waitcnt(0x0F70);  // (no copy may land after the workgroup has left)
    }
  } else {
    if (steps > 0) {
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the workgroup's own K, V rows are in (else the loop would wait for them each time round)
      DKV_LOAD(sq0, sd0, ps0, 0)
      DKV_LOAD(sq1, sd1, ps1, 1)
      DKV_STORE(sq0, sd0, ps0, 0)
      __syncthreads();
      for (int step = 0;; step += 2) {  // (every exit test is uniform over the workgroup)
        DKV_STEP(step, 2, 0, sq0, sd0, ps0, sq1, sd1, ps1)
        DKV_STEP(step + 1, 2, 1, sq1, sd1, ps1, sq0, sd0, ps0)
      }
    }
  }
#undef DKV_STEP
#undef DKV_LOAD
#undef DKV_STORE
  // Out through LDS, so that whole rows of 256 bytes leave at a time: a wavefront's 32 keys of dK, then of dV.
  __syncthreads();                       // (nobody reads the staging buffers, and no copy lands in them any more)
  constexpr int OP = 256 + 16;           // bytes per staged row
  static_assert(2 * KB * 32 * OP <= 2 * BUF_B, "a wavefront's rows fit");
  // (everything from the thread's number again: values of the prologue held for this through the loop took registers from
  // it, and at KB = 2, where it has none to spare, operand addresses went to scratch memory, whose reloads in the middle of
  // a step waited for the rows just requested: 12 heads x 32760 tokens, three quarters critical, backward pass 26.0 -> 24.2 ms)
  int te = t;
  if constexpr (KB == 2) asm volatile("" : "+v"(te));
  const int le = te & 63, we = te >> 6, l32e = le & 31, hfe = le >> 5;
  unsigned char* my = lds + we * 32 * OP;
  const int row0 = 64 * (KB * J + (KB == 2 ? we >> 1 : 0)) + 32 * (we & 1);
  auto store_rows = [&](const v16f (&x)[4], float scale, bf16_t* dst, const Layout& L) __attribute__((always_inline)) {
    bf16_t* to = slice_of(dst, L, bh, dm.H) + (row0 + (le >> 4)) * L.sn + (le & 15) * 8;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4)
        *(uint2*)(my + l32e * OP + (32 * ct + 8 * g4 + 4 * hfe) * 2) =
            uint2{pack_bf16x2(x[ct][4 * g4] * scale, x[ct][4 * g4 + 1] * scale), pack_bf16x2(x[ct][4 * g4 + 2] * scale, x[ct][4 * g4 + 3] * scale)};
    __builtin_amdgcn_wave_barrier();     // (a wavefront's LDS operations execute in order: only the compiler has to keep it)
    v4i out[8];
#pragma unroll
    for (int it = 0; it < 8; ++it) out[it] = *(const v4i*)(my + (4 * it + (le >> 4)) * OP + (le & 15) * 16);
    __builtin_amdgcn_wave_barrier();
    if (row0 + 32 <= dm.N) {             // (uniform)
#pragma unroll
      for (int it = 0; it < 8; ++it) __builtin_memcpy(to + 4 * it * L.sn, &out[it], 16);
    } else {
#pragma unroll
      for (int it = 0; it < 8; ++it)
        if (row0 + 4 * it + (le >> 4) < dm.N) __builtin_memcpy(to + 4 * it * L.sn, &out[it], 16);
    }
  };
  store_rows(dkt, DK_SIGN * INV_SQRT_D, dk, L_dk);
  store_rows(dvt, 1.0f, dv, L_dv);
}
template <int KB, int TILES, int PHI, bool ST = false>
__global__ void __launch_bounds__(128 * KB) bwd_dkv_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ dout,
                                                      const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                                      const int8_t* __restrict__ mask, const float* __restrict__ lse2,
                                                      const float* __restrict__ delta, const bf16_t* __restrict__ G,
                                                      bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int pair_shift,
                                                      const int* __restrict__ order, int natural, BwdDims dm) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  dkv_block<KB, TILES, PHI, ST>(q, dout, k, v, mask, lse2, delta, G, dk, dv, pair_shift, order, natural, dm, lds, blockIdx.x, gridDim.x);
}
// dK/dV and, in the workgroups behind theirs, dQ (two wavefronts of 32 query rows each), which needs nothing of it: for
// calls whose workgroups of either kind leave compute units empty or end one by one.
struct DqPart {
  const int32_t* crit;
  const float* dq_lin;
  bf16_t* dq;
  int first, per;                // number of the first workgroup of dQ; workgroups per query block
};
template <int PHI, bool ST>
__global__ void __launch_bounds__(128, 1) bwd_dq_dkv_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ dout,
                                                           const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                                           const int8_t* __restrict__ mask, const float* __restrict__ lse2,
                                                           const float* __restrict__ delta, const bf16_t* __restrict__ G,
                                                           bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int pair_shift,
                                                           const int* __restrict__ order, int natural, DqPart part, BwdDims dm) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int number = (int)blockIdx.x - part.first;
  if (number < 0) {
    dkv_block<1, 2, PHI, ST>(q, dout, k, v, mask, lse2, delta, G, dk, dv, pair_shift, order, natural, dm, lds, blockIdx.x, part.first);
  } else {
    int unit, bh;
    if (xcd_block(part.per * dm.Tq, unit, bh, number))
      dq_block<2, 1, ST>(q, dout, k, v, part.crit, lse2, delta, part.dq_lin, part.dq, dm, lds, unit, part.per, bh);
  }
}

// ---------------------------------------------------------------------------------------------
// Do all of these layouts equal the contiguous [B,H,N,d] one?  (Then the instances with compile-time strides serve.)
static bool contiguous(const Problem& p, std::initializer_list<const Layout*> ls) {
  const Layout c = contiguous_layout(p.H, p.N);
  for (const Layout* L : ls)
    if (L->sb != c.sb || L->sh != c.sh || L->sn != c.sn) return false;
  return true;
}

static BwdDims bwd_dims(const Problem& p) {
  return BwdDims{p.N, p.Tq, p.Tk, p.n_c, p.Tq * (p.block_q / 32), p.H, p.lq, p.lk, p.lv, p.ld, p.ldq, p.ldk, p.ldv, p.lo};
}

// The launchers below that return an int return 0, or -1 when the kernel's LDS allowance could not be set (then nothing
// is launched; the result of the attribute call is cached, the failure is reported on every call).
void launch_bwd_stats(const Problem& p, const void* q, const void* k, const void* v, const void* dout,
                     const int32_t* crit, float* lse2, float* delta, hipStream_t stream) {
  const unsigned grid = (unsigned)(8 * ((p.Tq + 7) / 8) * p.BH);
  const bool st = !contiguous(p, {&p.lq, &p.lk, &p.lv, &p.ld});
  // One tile per wavefront where two would leave SIMDs without a wavefront: the walk over a list is then the shorter
  // one (3 heads x 4617 tokens, query blocks of 64: 20.0 against 26.7 us; 14 heads 47 us, 72 before).
  const bool narrow = (long long)p.Tq * p.BH * (p.block_q / 64) < 1024;
#define SLA_STATS(WAVES, QT, ST) bwd_lse_delta_kernel<WAVES, QT, ST><<<grid, WAVES * 64, 0, stream>>>( \
      (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (const bf16_t*)dout, crit, lse2, delta, bwd_dims(p))
#define SLA_STATS_ST(WAVES, QT) { if (st) SLA_STATS(WAVES, QT, true); else SLA_STATS(WAVES, QT, false); }
  if (p.block_q == 128) {
    if (narrow) SLA_STATS_ST(4, 1) else SLA_STATS_ST(2, 2)
  } else {
    if (narrow) SLA_STATS_ST(2, 1) else SLA_STATS_ST(1, 2)
  }
#undef SLA_STATS_ST
#undef SLA_STATS
}

// The unquantised forward pass; with `codes`, the same on
// INT8 codes of Q and K (SLA_QUANT_QK_INT8: integer products, 16-bit P and V).
void launch_fwd_bf16(const Problem& p, const void* q, const void* k, const void* v, const int32_t* crit,
                    const bf16_t* HZ, const bf16_t* proj_b, int phi_kind, void* out, const SaveTo* save,
                    const CodeScales* codes, hipStream_t stream) {
  const unsigned grid = (unsigned)(8 * ((p.Tq + 7) / 8) * p.BH);
  const FwdEpilogue fe{HZ, HZ ? proj_b : nullptr, (bf16_t*)out, phi_kind, save ? save->lse2 : nullptr, save ? save->os : nullptr,
                       save ? save->hdr_dst : nullptr, save ? save->hdr : SavedHeader{},
                       codes ? codes->dq : nullptr, codes ? codes->dk : nullptr, codes ? (const bf16_t*)codes->q_lin : nullptr, p.lq};
  BwdDims dm = bwd_dims(p);
  if (codes) dm.lq = dm.lk = contiguous_layout(p.H, p.N);   // the code tensors are the library's own
  const bool st = codes ? !contiguous(p, {&p.lv, &p.lo}) : !contiguous(p, {&p.lq, &p.lk, &p.lv, &p.lo});
#define SLA_FWD16(NW, CODES, ST) fwd_bf16_kernel<NW, CODES, ST><<<grid, NW * 64, 0, stream>>>( \
      (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, crit, dm, fe)
#define SLA_FWD16_ST(NW, CODES) { if (st) SLA_FWD16(NW, CODES, true); else SLA_FWD16(NW, CODES, false); }
  if (p.block_q == 128) {
    if (codes) SLA_FWD16_ST(4, true) else SLA_FWD16_ST(4, false)
  } else {
    if (codes) SLA_FWD16_ST(2, true) else SLA_FWD16_ST(2, false)
  }
#undef SLA_FWD16_ST
#undef SLA_FWD16
}

__global__ void __launch_bounds__(256) bwd_delta_kernel(const DeltaArgs X) { delta_block(X, blockIdx.x); }

void launch_bwd_delta(const DeltaArgs& X, const Problem& p, hipStream_t stream) {
  bwd_delta_kernel<<<(unsigned)delta_blocks(p), 256, 0, stream>>>(X);
}

// One tile per wavefront where two would leave SIMDs without a wavefront (query blocks of 64, 4617 tokens, us before ->
// now: 3 heads 28.5 -> 27.2, 14 heads 93 -> 79 with one tile; 20 heads 126 -> 102 with two)
static bool dq_narrow(const Problem& p) { return (long long)p.Tq * p.BH * (p.block_q / 64) < 1024; }
// Two key blocks per workgroup halve the bytes streamed where their lists coincide and idle half
// a workgroup where they do not: worth it only when most blocks are critical (at the paper's
// 10-15 % the lists of neighbours share 60 % and one key block per workgroup is 25 % faster).
static bool dkv_paired(const Problem& p) { return 2 * p.n_c > p.Tk; }
// dQ with dK and dV in one launch: either kind alone leaves wavefronts' places empty or runs on with a few long lists, and
// neither needs anything of the other.  Backward pass in us, two launches / one: 4 x 2187 in blocks of 64 (140 workgroups each)
// 119 / 95, 3 x 4617 136 / 113, 12 x 4617 262 / 244, 8 x 1024 82 / 71, 40 x 1024 in blocks of 128 178 / 161, 7 x 4617 200 / 165,
// 1 x 37800 629 / 533, 3 x 16380 363 / 328 (10 % critical).  From 1024 wavefronts' worth of query rows on dQ's wavefronts own 64 rows
// each; an instance of that form here gained on a training step 4 % of 40 x 4617, 2 % of 8 x 16380, nothing from 3 x 32760 on and lost
// 1 % of 8 x 75600: not kept.
// Long lists are nearly of one length, and what counts is whether the workgroups of both kinds, two at a time on a compute unit,
// go round in fewer turns than those of each: they do where the last turn of either is at most half full.  From a saved state,
// us, with lists of 20, 35 and 50 % of the blocks.  512 workgroups of dQ: 1 x 32760 in blocks of 128 533 / 534, 760 / 781, 999 /
// 1016; 782: 1 x 50000 1156 / 1024, 1708 / 1736, 2417 / 2540; 876: 2 x 28000 in blocks of 64 698 / 698, 1083 / 1115, 1465 /
// 1530; 880: 4 x 14000 410 / 407, 596 / 614, 787 / 817; 938: 1 x 60000 1435 / 1399, 2250 / 2312, 3194 / 3323; but 256: 1 x 16380
// 319 / 258, 373 / 292, 432 / 319; 626: 1 x 40000 825 / 740, 1278 / 1164, 1802 / 1603; 628: 2 x 20000 479 / 416, 711 / 632, 966 /
// 850; and where each kind has one turn, of blocks of 64, whose K and V one launch streams no more often, 438: 1 x 28000 456 /
// 454, 644 / 644, 828 / 798, 512: 2 x 16380 at 20, 30 and 50 % 350 / 317, 415 / 404, 560 / 555, and of 128 up to a third of the
// blocks (one launch's time at 25, 30 and 50 %: 314, 1 x 20000 0.85, 0.91, 0.99; 376, 1 x 24000 0.95, 0.97, 1.02; 2 x 16380
// 0.95, 0.98, 1.02).  Up to 48 blocks a list's length does not settle it (852: 6 x 9000, 49 and 70 blocks 431 / 434 and 549 /
// 567; 426: 3 x 9000, 42 blocks 233 / 223).
bool bwd_dq_with_dkv(const Problem& p) {
  if (!dq_narrow(p) || dkv_paired(p)) return false;
  const int places = 2 * compute_units();
  const long long units = (long long)p.Tq * p.BH * (p.block_q / 64);
  return p.n_c <= 48 || 5 * p.n_c <= p.Tk || (units - 1) % places < places / 2 ||
         (units <= places && (p.block_q == 64 || 3 * p.n_c <= p.Tk));
}

void launch_bwd_dq(const Problem& p, const void* q, const void* dout, const void* k, const void* v, const int32_t* crit,
                  const float* lse2, const float* delta, const float* dq_lin, void* dq, hipStream_t stream) {
  const unsigned grid = (unsigned)(8 * ((p.Tq + 7) / 8) * p.BH);
  const bool st = !contiguous(p, {&p.lq, &p.lk, &p.lv, &p.ld, &p.ldq});
  const bool narrow = dq_narrow(p);
#define SLA_DQ(WAVES, QT, ST) bwd_dq_kernel<WAVES, QT, ST><<<grid, WAVES * 64, 0, stream>>>( \
      (const bf16_t*)q, (const bf16_t*)dout, (const bf16_t*)k, (const bf16_t*)v, crit, lse2, delta, dq_lin, (bf16_t*)dq, bwd_dims(p))
#define SLA_DQ_ST(WAVES, QT) { if (st) SLA_DQ(WAVES, QT, true); else SLA_DQ(WAVES, QT, false); }
  if (p.block_q == 128) {
    if (narrow) SLA_DQ_ST(4, 1) else SLA_DQ_ST(2, 2)
  } else {
    if (narrow) SLA_DQ_ST(2, 1) else SLA_DQ_ST(1, 2)
  }
#undef SLA_DQ_ST
#undef SLA_DQ
}

template <int PHI, bool ST>
static int launch_bwd_dkv_phi(const Problem& p, const void* q, const void* dout, const void* k, const void* v, const int8_t* mask,
                               const float* lse2, const float* delta, const bf16_t* G, void* dk, void* dv, int* order_ws, const DqWith* with, hipStream_t stream) {
  // dynamic LDS: two staging buffers, the rows' lse and delta, the list of query blocks
  const int list_bytes = (2 * p.Tq + 15) & ~15;
  const int lds2 = 2 * 4 * TILE_B + 2 * 2 * 64 * 4 + list_bytes;
  const int lds1 = 2 * 4 * SWZ_TILE_B + 2 * 2 * 64 * 4 + list_bytes;
  static const bool ok =
      hipFuncSetAttribute((const void*)bwd_dkv_kernel<2, 2, PHI, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) == hipSuccess &&
      hipFuncSetAttribute((const void*)bwd_dkv_kernel<1, 2, PHI, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) == hipSuccess &&
      hipFuncSetAttribute((const void*)bwd_dq_dkv_kernel<PHI, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) == hipSuccess;
  if (!ok) return -1;
  const int tiles = p.block_q / 32;  // of a query block: 2 or 4
  if (dkv_paired(p)) {
    const int pairs = (p.Tk + 1) / 2;
    bwd_dkv_kernel<2, 2, PHI, ST><<<(unsigned)(8 * ((pairs + 7) / 8) * p.BH), 256, lds2, stream>>>(
        (const bf16_t*)q, (const bf16_t*)dout, (const bf16_t*)k, (const bf16_t*)v, mask, lse2, delta, G,
        (bf16_t*)dk, (bf16_t*)dv, tiles == 4 ? 1 : 0, nullptr, 0, bwd_dims(p));
  } else {
    // An order only where workgroups wait for a place (two fit a compute unit), and only of the last heads, as many as
    // the memory-side cache holds Q and dO of: what counts is the end of the launch, and with all of 40 x 75600 tokens
    // under way at once 25.8 ms became 29.6.  Whole backward pass in us, without / with an order, heads x key blocks: 33 x 16
    // (528) 174.7 / 179.8, 13 x 40 (520) 174.8 / 174.3, 24 x 24 (576) 184.2 / 181.7, 12 x 48 (576) 185.8 / 182.4, 8 x 73 (584)
    // 241.5 / 238.3, 5 x 126 (630) 243.9 / 235.2, 12 x 73 (876) 246.7 / 234.6, 2 x 512 (1024) 611 / 528, 80 x 16 (1280) 313.9 /
    // 308.7, 12 x 126 (1512) 420 / 393, 24 x 512 (12288) 6283 / 6024, but 80 x 40 (3200) 671 / 678; 10 x 37, where none of the
    // 370 workgroups waits, 123.1 / 128.8.  Lists of one length, as white noise has them, gain nothing and pay the 5 to 10 us.
    const long long head_bytes = 4ll * p.N * D;
    const int heads = (int)std::min<long long>(p.BH, std::max<long long>(1, (224ll << 20) / head_bytes));
    const bool ordered = order_ws && p.BH * p.Tk > 2 * compute_units();
    const int first = ordered ? p.BH - heads : p.BH, total = heads * p.Tk, per = (total + 7) / 8;
    const int natural = 8 * ((p.Tk + 7) / 8) * first;
    int *counts = order_ws, *order = order_ws + total;
    if (ordered) {
      dkv_counts_kernel<<<(unsigned)(heads * ((p.Tk + 63) / 64)), 1024, 0, stream>>>(mask + (size_t)first * p.Tq * p.Tk, p.Tq, p.Tk, counts);
      dkv_order_kernel<<<8, 1024, 0, stream>>>(counts, total, per, first * p.Tk, order);
    }
    const unsigned grid = (unsigned)natural + (ordered ? 8u * (unsigned)per : 0u);
    if (with) {
      const int units = p.block_q / 64;
      const DqPart part{with->crit, with->dq_lin, (bf16_t*)with->dq, (int)grid, units};
      bwd_dq_dkv_kernel<PHI, ST><<<grid + (unsigned)(8 * ((units * p.Tq + 7) / 8) * p.BH), 128, lds1, stream>>>(
          (const bf16_t*)q, (const bf16_t*)dout, (const bf16_t*)k, (const bf16_t*)v, mask, lse2, delta, G,
          (bf16_t*)dk, (bf16_t*)dv, tiles == 4 ? 1 : 0, order, natural, part, bwd_dims(p));
      return 0;
    }
    bwd_dkv_kernel<1, 2, PHI, ST><<<grid, 128, lds1, stream>>>(
        (const bf16_t*)q, (const bf16_t*)dout, (const bf16_t*)k, (const bf16_t*)v, mask, lse2, delta, G,
        (bf16_t*)dk, (bf16_t*)dv, tiles == 4 ? 1 : 0, order, natural, bwd_dims(p));
  }
  return 0;
}

// (the feature map matters to the prologue only -- the linear branch's share -- and only when G is given)
int launch_bwd_dkv(const Problem& p, const void* q, const void* dout, const void* k, const void* v, const int8_t* mask,
                   const float* lse2, const float* delta, const bf16_t* G, int phi_kind, void* dk, void* dv, int* order_ws, const DqWith* with, hipStream_t stream) {
  const int phi = G ? phi_kind : 0;
  const bool st = !contiguous(p, {&p.lq, &p.lk, &p.lv, &p.ld, &p.ldk, &p.ldv}) || (with && !contiguous(p, {&p.ldq}));
#define SLA_DKV(PHI) (st ? launch_bwd_dkv_phi<PHI, true>(p, q, dout, k, v, mask, lse2, delta, G, dk, dv, order_ws, with, stream) \
                         : launch_bwd_dkv_phi<PHI, false>(p, q, dout, k, v, mask, lse2, delta, G, dk, dv, order_ws, with, stream))
  return phi == 0 ? SLA_DKV(0) : phi == 1 ? SLA_DKV(1) : SLA_DKV(2);
#undef SLA_DKV
}

}  // namespace sla
