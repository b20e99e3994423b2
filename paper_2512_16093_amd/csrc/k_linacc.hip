// lin_accumulate: per query block, the sums of the marginal key blocks' summaries,
//     HZ[i][n] = sum_{j : block j marginal for i} hz[j][n],   n over the 129*128 entries
// of a summary (h'^T and the z row), written as one dense contraction per (b,h):
//     HZ[Tq x 16512] = M0[Tq x Tk] . hz[Tk x 16512],   M0 = 1 where the mask is 0.
// This really is a GEMM (every summary is needed by ~n_m/Tk of all query blocks), so it
// runs on bf16 MFMA with fp32 accumulation; gathering n_m summaries per query block
// instead would move ~50x more bytes.
//
// The two operands could not be more different: hz is the big one (tens of MB per head) and
// M0 is a bit matrix.  So a workgroup owns a 128-column stripe of hz for 384 query blocks at
// once, the (few) row chunks of a stripe run at the same time on one XCD so that hz comes
// from HBM once, and M0 travels as bits: one 32-bit word per (query block,
// tile of 32 key blocks), 3 KiB per staged tile against 8 KiB of hz.  The bf16 A operand of a
// wavefront is made from its mask byte through a 256-entry table in LDS (entry b = the eight
// bf16 values 0.0 / 1.0 of the bits of b), one 16-byte LDS read per fragment (two reads of a 16-entry
// table whose entries never meet in a bank: 2 to 6 % slower).
//
// Workgroup = 4 wavefronts, two workgroups per CU (independent, so the two wavefronts of a
// SIMD are not in step); in a full chunk wavefront w owns query blocks [96 w, 96 w + 96) x 128
// columns (3 x 4 MFMA tiles of 32 x 32, 192 accumulator registers); a head's shorter last chunk
// is dealt to the wavefronts in even runs of row tiles and runs a copy of the loop with fewer
// tiles per wavefront.  Tiles are accumulated transposed (the hz fragment is the MFMA's A
// operand) so that a lane ends up with runs of consecutive entries of one query block's
// summary, which leave through LDS as whole lines.  Operand tiles for 64 key blocks at a time are
// copied global -> LDS asynchronously, three stages deep (one barrier per tile).  hz rows are copied
// as they are (n contiguous) and read back with the LDS transposing read of gfx950
// (ds_read_b64_tr_b16): the contraction index j is the slow index of hz, so one transposition
// is unavoidable, and this one costs 8 LDS reads per 12 MFMAs and no vector-ALU work.
#include <algorithm>
#include <type_traits>

#include "reduce.h"

namespace sla {

constexpr int LA_KSUB = 2;                       // 32-block groups per staged tile
constexpr int LA_KT = 32 * LA_KSUB;              // key blocks per staged tile (one barrier per tile)
constexpr int LA_ROWS = 384, LA_COLS = 128;      // workgroup tile
constexpr int LA_WAVES = 4;
constexpr int LA_M_ROWS = 512;                   // mask words staged per 32-block group (two 1 KiB pieces; 384 used)
constexpr int LA_B_ROW = LA_COLS * 2;            // 256 bytes per staged hz row
// A row's sixteen 16-byte chunks are staged permuted, chunk c of row r at position c ^ la_swz(r): the 16 lanes of a transposing
// read's group address four rows, which at 256 bytes apart met in the same banks: 222 of the LDS's 321 M cycles of 40 slices of 591 x
// 1182 blocks were conflicts, now 71 of 170 M, and nearly all of those are of the table, whose entries meet at random (9 M with one
// entry read always).  There 897 us, now 812, of 1182 x 1182 1793 / 1590, 12 of 256 x 512 70.4 / 67.0.
__device__ __forceinline__ int la_swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
constexpr int LA_B_BYTES = LA_KT * LA_B_ROW;
constexpr int LA_OUT_PITCH = 64 * 2 + 16;         // bytes per row of 64 results on their way out
constexpr int LA_B_STAGE = ((LA_B_BYTES > LA_WAVES * 32 * LA_OUT_PITCH ? LA_B_BYTES : LA_WAVES * 32 * LA_OUT_PITCH) + 255) / 256 * 256;
constexpr int LA_M_PIECES = 2 * LA_KSUB;         // 1 KiB pieces of mask words per tile
static_assert(HZ_ELEMS % LA_COLS == 0, "the stripes tile a summary exactly");
static_assert(LA_M_PIECES == LA_WAVES && 8 * LA_KSUB % LA_WAVES == 0, "every wavefront copies the same number of pieces");

__host__ __device__ inline int la_k_tiles(int Tk) { return (Tk + 31) / 32; }  // word columns of the bit matrix
__host__ __device__ inline int la_row_chunks(int Tq) { return (Tq + LA_ROWS - 1) / LA_ROWS; }
// row stride of the bit matrix: the chunks, plus the slack the last chunk's 512-word copies run into
__host__ __device__ inline int la_rows_padded(int Tq) { return la_row_chunks(Tq) * LA_ROWS + (LA_M_ROWS - LA_ROWS); }

// mbits[bh][kt][i] (kt < ceil(Tk/32), i < la_rows_padded(Tq)): bit e = 1 where key block 32 kt + e is marginal
// for query block i.  Words of rows >= Tq are never written and never matter (their results
// are not stored); bits of key blocks >= Tk are 0.
__global__ void marginal_bits_kernel(const int8_t* __restrict__ mask, int Tq, int Tk, int BH,
                                     uint32_t* __restrict__ mbits) {
  const int KT = la_k_tiles(Tk), TqP = la_rows_padded(Tq);
  const size_t total = (size_t)BH * KT * Tq;
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < total; x += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(x % Tq), kt = (int)((x / Tq) % KT), bh = (int)(x / ((size_t)Tq * KT));
    const int8_t* src = mask + ((size_t)bh * Tq + i) * Tk;
    uint32_t w = 0;
    for (int e = 0; e < 32; ++e) {
      const int j = kt * 32 + e;
      if (j < Tk && src[j] == 0) w |= 1u << e;
    }
    mbits[((size_t)bh * KT + kt) * TqP + i] = w;
  }
}

typedef __attribute__((address_space(3))) void* la_lds_ptr_t;

// Asynchronous 16-bytes-per-lane copy global -> LDS: lane l reads base + voff and the data lands
// at LDS address lds + 16 l.  Written as inline assembly on purpose: the compiler then neither
// knows nor cares that copies are in flight (it would otherwise make every LDS read it cannot
// prove disjoint wait for ALL of them); the pipeline below waits for them by explicit counts.
// Loads the compiler does not know about only make its own waits more conservative.
__device__ __forceinline__ void la_copy16(const void* base, unsigned voff, const void* lds) {
  const unsigned lds_addr = (unsigned)(uintptr_t)(la_lds_ptr_t)lds;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
               :
               : "s"(base), "v"(voff), "s"(lds_addr)
               : "memory", "m0");
}

// LDS read with transposition (16-bit elements): in every group of 16 lanes, lane i receives, for
// e = 0..3, element i % 4 of the 8 bytes addressed by lane 4 e + i / 4 of the group.  With lane
// s of a group addressing row s / 4, columns 4 (s % 4) .. +3 of a 4-row x 16-column patch, lane
// i ends up with the four rows of column i: a k-contiguous MFMA operand out of a row-major tile.
typedef short v4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4s la_read_tr(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p);
}

__device__ __forceinline__ void la_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The same bit matrix for the transposed mask (backward pass: sums over the query blocks that hold a key block as
// marginal): mbits_t[bh][qt][j] (qt < ceil(Tq/32), j < la_rows_padded(Tk)): bit e = 1 where key block j is marginal for
// query block 32 qt + e.  A wavefront transposes 64 query blocks x 32 key blocks by ballots; from the int8 mask,
// byte by byte, it was a launch of 37 us at 40 slices of 591 x 1182 blocks and of 8 at 4 of 35 x 35.
__device__ __forceinline__ void transpose_bits(const uint32_t* __restrict__ mbits, int Tq, int Tk, int BH, uint32_t* __restrict__ mbits_t,
                                               int blk, int blocks) {
  const int KT = la_k_tiles(Tk), TqP = la_rows_padded(Tq), QT = la_k_tiles(Tq), TkP = la_rows_padded(Tk), Q64 = (Tq + 63) / 64;
  const int lane = threadIdx.x & 63;
  const unsigned total = (unsigned)BH * KT * Q64;
  for (unsigned x = blk * LA_WAVES + (threadIdx.x >> 6); x < total; x += blocks * LA_WAVES) {
    const int bk = (int)(x / (unsigned)Q64), q64 = (int)(x - (unsigned)bk * Q64), bh = bk / KT, kt = bk - bh * KT;
    const int i = 64 * q64 + lane;
    const uint32_t word = i < Tq ? mbits[((size_t)bh * KT + kt) * TqP + i] : 0u;
    uint32_t out = 0;
#pragma unroll 4   // (all 32 at once would take every scalar register)
    for (int b = 0; b < 32; ++b) {
      const unsigned long long col = __ballot((word >> b) & 1u);
      const uint32_t half = lane < 32 ? (uint32_t)col : (uint32_t)(col >> 32);
      if ((lane & 31) == b) out = half;
    }
    const int qt = 2 * q64 + (lane >> 5);
    if (qt < QT) mbits_t[((size_t)bh * QT + qt) * TkP + 32 * kt + (lane & 31)] = out;
  }
}

// (RIDERS: an instance of its own: one for both spilled registers and made short forward calls 2 to 4 % slower)
template <bool RIDERS>
__global__ void __launch_bounds__(LA_WAVES * 64, 2) lin_accumulate_kernel(const uint32_t* __restrict__ mbits,
                                                                          const bf16_t* __restrict__ hz, int Tq, int Tk,
                                                                          int groups, bf16_t* __restrict__ HZ, int rider_blocks, int BH, LinRiders riders) {
  // three stages, each a tile of hz rows and the mask words that go with it; separate objects,
  // so the compiler can tell the asynchronous fill of one stage from the reads of another
  __shared__ __attribute__((aligned(1024))) unsigned char hz0[LA_B_STAGE], hz1[LA_B_STAGE], hz2[LA_B_STAGE];
  __shared__ __attribute__((aligned(1024))) uint32_t mw0[LA_KSUB * LA_M_ROWS], mw1[LA_KSUB * LA_M_ROWS], mw2[LA_KSUB * LA_M_ROWS];
  __shared__ uint4 lut[256];
  const int t = threadIdx.x, lane = t & 63, l32 = lane & 31, hf = lane >> 5;
  if (RIDERS && (int)blockIdx.x < rider_blocks) {  // (the small work in front, LinRiders)
    if (riders.mbits_t) transpose_bits(mbits, Tq, Tk, BH, riders.mbits_t, blockIdx.x, rider_blocks);
    else reduce_block(riders.reduce, blockIdx.x, (float4(*)[16])hz0);
    return;
  }
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int KT32 = la_k_tiles(Tk), KT = (KT32 + LA_KSUB - 1) / LA_KSUB, TqP = la_rows_padded(Tq);
  constexpr int STRIPES = HZ_ELEMS / LA_COLS;
  const int chunks = la_row_chunks(Tq);

  {  // table: mask byte -> eight bf16 0.0 / 1.0 (256 threads = 256 entries)
    uint32_t x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x[e] = ((t >> (2 * e)) & 1 ? 0x3f80u : 0u) | ((t >> (2 * e + 1)) & 1 ? 0x3f800000u : 0u);
    lut[t] = make_uint4(x[0], x[1], x[2], x[3]);
  }

  const unsigned lane16 = (unsigned)lane * 16u;
  // this lane's address inside a B patch for the transposing reads: lane group g = lane / 16
  // serves columns 16 (g % 2) .. +15 and staged rows 8 (g / 2) + (0..3) [+ 4 for the second read, whose chunks are
  // permuted by one more]; the column tile is flipped into the address
  const int tr_row = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int tr_off = tr_row * LA_B_ROW + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ la_swz(tr_row)) << 4) + 8 * (lane & 1);
  __syncthreads();  // publishes the table

  // Persistent workgroups, two per compute unit: each takes work items (b,h, stripe, row chunk)
  // in turn.  The row chunks of one stripe are consecutive items, and consecutive items go to
  // workgroups of the same XCD (workgroup ids are dealt round-robin over the 8 XCDs), so the
  // chunks of a stripe run at the same time on one L2 and the stripe comes from HBM once.  The
  // stripes of one head run next to each other in time (they share the head's mask words).
  // An item's first two tiles are requested before the results of the item before it are stored, so that its loop does
  // not begin with a wait for memory: with that and whole-line stores (below) 40 slices of 591 x 1182 blocks went from 1037 to
  // 870 us, 40 of 1182 x 1182 from 2008 to 1750, 12 of 256 x 512 from 93 to 70 (shorter chunks of rows there: the
  // stripes are read more often than idle slots are saved, 427 -> 441 us for the whole call).
  if constexpr (!RIDERS) rider_blocks = 0;
  const int wg = blockIdx.x - rider_blocks;                          // (rider_blocks and the rest are multiples of 8)
  const int xcd = wg & 7, slot = wg >> 3, slots = (gridDim.x - rider_blocks) >> 3;
  // (groups: (b,h, stripe) pairs; group g runs on XCD g % 8)
  // Slot s takes, of its XCD's groups one after another, the chunks s, s + slots, ...; in a group the chunks are rotated by
  // one for every round of the slots (a head's last chunk is usually shorter, and every workgroup should get its share of
  // short ones).  All of it is carried from item to item: found by divisions it took a microsecond per item.
  const int round_groups = max(1, slots / chunks), step_groups = slots / chunks, step_chunks = slots - step_groups * chunks;
  int grp = slot / chunks, place = slot - grp * chunks;            // group of this XCD, place in it
  int rot = grp / round_groups, in_round = grp - rot * round_groups;
  rot %= chunks;
  int bh = (grp * 8 + xcd) / STRIPES, stripe = grp * 8 + xcd - bh * STRIPES;
  int row0 = 0, n0 = 0;
  const char *hz_bh, *mb_bh;     // uniform: the item's stripe and its mask words
  auto enter = [&]() {
    const int chunk = place + rot >= chunks ? place + rot - chunks : place + rot;
    n0 = stripe * LA_COLS;
    row0 = chunk * LA_ROWS;
    hz_bh = (const char*)(hz + (size_t)bh * Tk * HZ_ELEMS + n0);
    mb_bh = (const char*)(mbits + (size_t)bh * KT32 * TqP + row0);
  };
  auto advance = [&]() {
    int by = step_groups;
    place += step_chunks;
    if (place >= chunks) { place -= chunks; ++by; }
    grp += by;
    in_round += by;
    for (; in_round >= round_groups; in_round -= round_groups) rot = rot + 1 == chunks ? 0 : rot + 1;
    for (stripe += 8 * by; stripe >= STRIPES; stripe -= STRIPES) ++bh;
  };
  // asynchronous copy of tile kt into a stage, in 1 KiB pieces (4 hz rows, or 256 mask words)
  // dealt round-robin to the wavefronts
  auto fetch = [&](int kt, unsigned char* hzs, uint32_t* mws) {
#pragma unroll
    for (int u = 0; u < 8 * LA_KSUB / LA_WAVES; ++u) {
      const int p = w + LA_WAVES * u;
      const int r = 4 * p + (lane >> 4), j = min(kt * LA_KT + r, Tk - 1);  // rows past Tk repeat the last one (their mask bits are 0)
      const unsigned off = (unsigned)j * (unsigned)(HZ_ELEMS * 2) + (unsigned)((lane & 15) ^ la_swz(r)) * 16u;
      la_copy16(hz_bh, off, hzs + p * 1024);
    }
    {
      const int sub = w >> 1, part = w & 1;  // one mask piece per wavefront
      const int kt32 = min(kt * LA_KSUB + sub, KT32 - 1);  // (a word column past the end is ignored by the consumer)
      la_copy16(mb_bh + ((size_t)kt32 * TqP + 256 * part) * 4, lane16, mws + sub * LA_M_ROWS + part * 256);
    }
  };
  // copies of a wavefront per tile, and the wait that leaves at most one tile's worth in flight
  constexpr int PER_TILE = 8 * LA_KSUB / LA_WAVES + 1;
  static_assert(PER_TILE <= 15, "wait count immediate");
  auto wait_keep = [&](bool keep_one) {
    if (keep_one) __builtin_amdgcn_s_waitcnt(0x0F70 | PER_TILE);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
  };
  auto fetch_first = [&]() {
    fetch(0, hz0, mw0);
    if (KT > 1) fetch(1, hz1, mw1);
  };

  // The first tile's copies are followed by the second tile's and by the previous item's `stored` stores, and vector
  // memory operations complete in order: all but that many may stay in flight (rounded down to what the switch names).
  int stored = 0;
  auto wait_first = [&]() {
#define LA_WAIT(N) { if (KT > 1) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N + PER_TILE) : "memory"); else asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
    if (stored >= 24) LA_WAIT(24) else if (stored >= 16) LA_WAIT(16) else if (stored >= 8) LA_WAIT(8) else if (stored >= 2) LA_WAIT(2) else LA_WAIT(0)
#undef LA_WAIT
  };

  if (grp * 8 + xcd >= groups) return;  // (uniform)
  enter();
  fetch_first();
  while (grp * 8 + xcd < groups) {
  // The chunk's row tiles (of 32 query blocks; 12 in a full chunk, fewer in a head's last one)
  // are dealt to the four wavefronts as evenly as consecutive runs allow, and the loop below is
  // instantiated for the largest share, so a short last chunk costs its share of MFMAs only.
  const int tiles_c = min(LA_ROWS / 32, (Tq - row0 + 31) / 32);
  const int t_base = tiles_c >> 2, t_rem = tiles_c & 3;
  const int my_tiles = t_base + (w < t_rem ? 1 : 0), wrow = 32 * (w * t_base + min(w, t_rem));
  auto run_item = [&](auto nmt_tag) {
  constexpr int NMT = decltype(nmt_tag)::value;
  v16f acc[NMT][4];
#pragma unroll
  for (int a = 0; a < NMT; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = v16f{};

#define LA_COMPUTE(KTI, HZS, MWS)                                                                         \
  _Pragma("unroll") for (int sub = 0; sub < LA_KSUB; ++sub) {                                             \
    uint32_t mw[NMT];                                                                                     \
    const bool live = (KTI) * LA_KSUB + sub < KT32; /* uniform: the last tile may be partly past the end */ \
    _Pragma("unroll") for (int mt = 0; mt < NMT; ++mt)                                                    \
      mw[mt] = live ? MWS[sub * LA_M_ROWS + wrow + 32 * mt + l32] : 0u;                                   \
    _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {                                                    \
      v8bf aop[NMT], bop[4];                                                                              \
      _Pragma("unroll") for (int mt = 0; mt < NMT; ++mt) {                                                \
        union { uint4 u; v8bf v; } c;                                                                     \
        c.u = lut[(mw[mt] >> (16 * ks + 8 * hf)) & 0xffu];                                                \
        aop[mt] = c.v;                                                                                    \
      }                                                                                                   \
      _Pragma("unroll") for (int nt = 0; nt < 4; ++nt) {                                                  \
        /* staged rows r0 + 8 hf + (0..7) of column 32 nt + l32, by two transposing reads */              \
        union { v4s h[2]; v8bf v; } u;                                                                    \
        const int r0 = 32 * sub + 16 * ks;                                                                \
        u.h[0] = la_read_tr(&HZS[(tr_off ^ (nt << 6)) + r0 * LA_B_ROW]);                                  \
        u.h[1] = la_read_tr(&HZS[(tr_off ^ (nt << 6) ^ 16) + (r0 + 4) * LA_B_ROW]);                       \
        bop[nt] = u.v;                                                                                    \
      }                                                                                                   \
      _Pragma("unroll") for (int mt = 0; mt < NMT; ++mt)                                                  \
        _Pragma("unroll") for (int nt = 0; nt < 4; ++nt)                                                  \
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bop[nt], aop[mt], acc[mt][nt], 0, 0, 0);  \
    }                                                                                                     \
  }

#define LA_STEP(KTI, HC, MC, HF, MF)           \
  {                                            \
    const int kt_ = (KTI);                     \
    if (kt_ + 2 < KT) fetch(kt_ + 2, HF, MF);  \
    LA_COMPUTE(kt_, HC, MC)                    \
    wait_keep(kt_ + 2 < KT);                   \
    la_barrier();                              \
  }
  wait_first();
  la_barrier();
  int kt = 0;
  for (; kt + 3 <= KT; kt += 3) {
    LA_STEP(kt, hz0, mw0, hz2, mw2)
    LA_STEP(kt + 1, hz1, mw1, hz0, mw0)
    LA_STEP(kt + 2, hz2, mw2, hz1, mw1)
  }
  if (kt < KT) LA_STEP(kt, hz0, mw0, hz2, mw2)
  if (kt + 1 < KT) LA_STEP(kt + 1, hz1, mw1, hz0, mw0)
#undef LA_STEP
#undef LA_COMPUTE
  // (no copy is in flight and every wavefront is done with the stages)

  // The tiles were accumulated transposed (summary entries along the MFMA rows, query blocks
  // along its columns), so a lane owns ONE query block and runs of 4 consecutive entries of
  // its summary.  They leave through the wavefront's quarter of stage 2, 32 rows of 64 entries at a time, as whole
  // 128-byte lines.
  // (a wavefront with fewer row tiles than NMT has accumulated a neighbour's rows in the spare
  // tiles; it does not store them)
  const int first_row = row0 + wrow, rows = min(32 * my_tiles, Tq - first_row);   // this wavefront's (none: <= 0)
  char* const out = (char*)(HZ + ((size_t)bh * Tq + first_row) * HZ_ELEMS + n0);  // uniform
  advance();
  if (grp * 8 + xcd < groups) {
    enter();
    fetch_first();
  }
  unsigned ln = lane;
  asm volatile("" : "+v"(ln));   // (the addresses below are formed per item: kept through the loop they cost registers that it has not got)
  unsigned char* const mine = hz2 + w * (32 * LA_OUT_PITCH);
  const unsigned out_off = (ln >> 3) * (unsigned)(HZ_ELEMS * 2) + (ln & 7) * 16u;
  unsigned char* const put = mine + (ln & 31) * LA_OUT_PITCH + (ln >> 5) * 8;
  const unsigned char* const get = mine + (ln >> 3) * LA_OUT_PITCH + (ln & 7) * 16;
#pragma unroll
  for (int mt = 0; mt < NMT; ++mt) {
    if (32 * mt >= rows) break;  // (uniform)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int n2 = 0; n2 < 2; ++n2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const v16f& a = acc[mt][2 * half + n2];
          *(uint2*)(put + (32 * n2 + 8 * g) * 2) =
              make_uint2(pack_bf16x2(a[4 * g], a[4 * g + 1]), pack_bf16x2(a[4 * g + 2], a[4 * g + 3]));
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (one wavefront's own region: its writes are done, no barrier)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 32 * mt + 8 * u;
        if (r >= rows) break;      // (uniform: a store that is issued has at least one row, which `stored` counts on)
        const uint4 v = *(const uint4*)(get + 8 * u * LA_OUT_PITCH);
        if (r + (int)(ln >> 3) < rows) *(uint4*)(out + (size_t)r * (HZ_ELEMS * 2) + 128 * half + out_off) = v;
      }
      asm volatile("" ::: "memory");
    }
  }
  stored = rows > 0 ? 2 * ((rows + 7) >> 3) : 0;
  };  // run_item
  const int nmt_item = t_base + (t_rem ? 1 : 0);
  if (nmt_item == 3) run_item(std::integral_constant<int, 3>{});
  else if (nmt_item == 2) run_item(std::integral_constant<int, 2>{});
  else run_item(std::integral_constant<int, 1>{});
  }  // work items
}

// The same sums for short heads (at most LS_MAX_ROWS query blocks and LS_MAX_KEYS key blocks): there a stripe is one or two staged
// tiles, and the kernel above waits for memory at every item, with three barriers around two dozen products.  Here
// nothing is staged: a wavefront takes 64 columns of all key blocks straight to registers, one dword (two adjacent columns)
// per lane and row, and makes of eight rows' dwords the operands of two products, one of the even columns and one of
// the odd; requested again for its next 64 columns as soon as they are consumed, so that a compute unit has up to 100 KB
// under way without a barrier.  The mask operands of its 32 RT query blocks are made once per head.  The contraction goes in
// the same steps in the same order (same bits).  A lane ends up with eight consecutive entries of a query block's summary:
// 16-byte stores, the lane halves' side by side.  Bound by memory: 24 slices of 37 x 73 blocks 29.8 -> 22.1 us (87 MB), 4 of
// 35 x 35 7.6 -> 6.4, 2 of 16 x 16 4.4 -> 3.4.
// Where the line lies (slices of query x key blocks, whole forward calls in us, staged / this): 40 of 16 x 16 59.7 / 49.5, of 8 x
// 16 57.8 / 45.9, of 32 x 64 163.0 / 156.7, 2 of 16 x 16 25.8 / 24.9, 24 of 37 x 73 112.6 / 110.0, 6 of 35 x 70 51.0 / 49.6, 3 of 40 x 80
// 44.0 / 43.6; but (in an instance for more) 40 of 48 x 96 269.7 / 270.4, 24 of 56 x 112 202.6 / 206.9, 40 of 64 x 64 187.2 / 194.8.  Above
// 32 query blocks, where the second product's rows are up to half empty, forward calls are within 2 % of each other whichever it is: 1 of 40
// x 80 38.9 / 39.4, 28 of 40 x 40 84.2 / 82.9, 40 of 48 x 48 122.3 / 122.9 (12 of 48 x 48, 780 workgroups' worth in 768 places, 50.5 /
// 53.7); staged where that alone was faster (33 to 48 query blocks of few slices) a training step of 4 of 35 x 35 took 1 % longer.
constexpr int LS_MAX_ROWS = 48, LS_MAX_KEYS = 80;
constexpr int LS_COLS = 64;
constexpr int ls_waves(int ksteps, int rt) { return ksteps == 4 || rt == 1 ? 3 : 2; }   // wavefronts per SIMD that its registers leave room for
static_assert(HZ_ELEMS % LS_COLS == 0, "64 columns at a time");
template <int KSTEPS, int RT, bool RIDERS>
__global__ void __launch_bounds__(256, ls_waves(KSTEPS, RT)) lin_short_kernel(const uint32_t* __restrict__ mbits, const bf16_t* __restrict__ hz, int Tq, int Tk,
                                                           int BH, bf16_t* __restrict__ HZ, int rider_blocks, LinRiders riders) {
  const int t = threadIdx.x, lane = t & 63, l32 = lane & 31, hf = lane >> 5, w = __builtin_amdgcn_readfirstlane(t >> 6);
  if constexpr (RIDERS) {
    __shared__ float4 sums[16][16];
    if ((int)blockIdx.x < rider_blocks) {
      if (riders.mbits_t) transpose_bits(mbits, Tq, Tk, BH, riders.mbits_t, blockIdx.x, rider_blocks);
      else reduce_block(riders.reduce, blockIdx.x, sums);
      return;
    }
  } else {
    rider_blocks = 0;
  }
  constexpr int GROUPS = HZ_ELEMS / LS_COLS, QUADS = (GROUPS + 3) / 4;   // of four wavefronts side by side
  const int KT32 = la_k_tiles(Tk), TqP = la_rows_padded(Tq);
  const int total = BH * QUADS, wg = blockIdx.x - rider_blocks, wgs = gridDim.x - rider_blocks;
  const int first = (int)((long long)total * wg / wgs), end = (int)((long long)total * (wg + 1) / wgs);
  const unsigned lane_off = (unsigned)(8 * hf * (HZ_ELEMS * 2) + 4 * l32);
  uint32_t x[KSTEPS][8];             // rows 16 ks + 8 hf + m of the columns under way
  v8bf mask[RT][KSTEPS];
  auto column = [&](int item) { return min(4 * (item % QUADS) + w, GROUPS - 1); };   // (past the end the last one again, not stored)
  auto request = [&](int item, int ks) __attribute__((always_inline)) {
    const char* from = (const char*)(hz + (size_t)(item / QUADS) * Tk * HZ_ELEMS) + column(item) * (LS_COLS * 2);
    // (the addresses are formed per load, a row's in scalar registers: as loop invariants they took 64 vector registers)
    if (16 * ks + 16 <= Tk) {        // (uniform)
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const char* row = from + (size_t)(16 * ks + m) * (HZ_ELEMS * 2);
        asm volatile("" : "+s"(row));
        x[ks][m] = *(const uint32_t*)(row + lane_off);
      }
    } else {                         // (rows past Tk repeat the last one: their mask bits are 0)
      int first_row = 16 * ks + 8 * hf;
      asm volatile("" : "+v"(first_row));
#pragma unroll
      for (int m = 0; m < 8; ++m) x[ks][m] = *(const uint32_t*)(from + ((unsigned)min(first_row + m, Tk - 1) * (unsigned)(HZ_ELEMS * 2) + 4u * l32));
    }
  };
  int have = -1;                     // whose mask operands these are
  if (first < end) {
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
      if (16 * ks < Tk) request(first, ks);
  }
  for (int item = first; item < end; ++item) {
    const int bh = item / QUADS;
    if (bh != have) {                // (uniform)
      have = bh;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const uint32_t* words = mbits + (size_t)bh * KT32 * TqP + 32 * rt + l32;
#pragma unroll
        for (int k2 = 0; k2 < KSTEPS / 2; ++k2) {
          const uint32_t word = 32 * k2 < Tk ? words[(size_t)k2 * TqP] : 0u;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t byte = word >> (16 * h + 8 * hf);
            union { uint32_t u[4]; v8bf v; } b;
#pragma unroll
            for (int e = 0; e < 4; ++e) b.u[e] = ((byte >> (2 * e)) & 1u) * 0x3f80u + ((byte >> (2 * e + 1)) & 1u) * 0x3f800000u;
            mask[rt][2 * k2 + h] = b.v;
          }
        }
      }
    }
    v16f acc[RT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[rt][0] = acc[rt][1] = v16f{};
    const int next = min(item + 1, end - 1);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      if (16 * ks >= Tk) break;      // (uniform)
      union { uint32_t u[4]; v8bf v; } even, odd;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        even.u[e] = __builtin_amdgcn_perm(x[ks][2 * e + 1], x[ks][2 * e], 0x05040100u);
        odd.u[e] = __builtin_amdgcn_perm(x[ks][2 * e + 1], x[ks][2 * e], 0x07060302u);
      }
      request(next, ks);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        acc[rt][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(even.v, mask[rt][ks], acc[rt][0], 0, 0, 0);
        acc[rt][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(odd.v, mask[rt][ks], acc[rt][1], 0, 0, 0);
      }
    }
    if (4 * (item - bh * QUADS) + w < GROUPS) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int row = 32 * rt + l32;
        if (row >= Tq) continue;
        char* dst = (char*)(HZ + ((size_t)bh * Tq + row) * HZ_ELEMS) + column(item) * (LS_COLS * 2) + 16 * hf;
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(uint4*)(dst + 32 * g) = uint4{pack_bf16x2(acc[rt][0][4 * g], acc[rt][1][4 * g]), pack_bf16x2(acc[rt][0][4 * g + 1], acc[rt][1][4 * g + 1]),
                                          pack_bf16x2(acc[rt][0][4 * g + 2], acc[rt][1][4 * g + 2]), pack_bf16x2(acc[rt][0][4 * g + 3], acc[rt][1][4 * g + 3])};
      }
    }
  }
}

size_t marginal_bits_t_bytes(const Problem& p) {
  return (size_t)p.BH * la_k_tiles(p.Tq) * la_rows_padded(p.Tk) * 4;
}

size_t marginal_bits_bytes(const Problem& p) {
  return (size_t)p.BH * la_k_tiles(p.Tk) * la_rows_padded(p.Tq) * 4;
}

void launch_marginal_bits(const Problem& p, const int8_t* mask, uint32_t* mbits, hipStream_t stream) {
  const size_t total = (size_t)p.BH * la_k_tiles(p.Tk) * p.Tq;
  const size_t want = (total + 255) / 256;
  const unsigned grid = (unsigned)(want < 1048560 ? want : 1048560);
  marginal_bits_kernel<<<grid, 256, 0, stream>>>(mask, p.Tq, p.Tk, p.BH, mbits);
}

void launch_lin_accumulate(const Problem& p, const uint32_t* mbits, const bf16_t* hz, bf16_t* HZ, const LinRiders& riders,
                           hipStream_t stream) {
  const int groups = (HZ_ELEMS / LA_COLS) * p.BH;
  // two workgroups per compute unit (192 accumulator registers per lane); a multiple of 8 (see the item order in the kernel)
  int grid = 2 * compute_units() / 8 * 8;
  if (grid < 8) grid = 8;
  // (at most 128 workgroups of the transposition: a quarter of the slots for 8 us at 40 slices of 591 x 1182 blocks)
  int rb = 0;
  if (riders.mbits_t) rb = (int)std::min<long long>(128, ((long long)p.BH * la_k_tiles(p.Tk) * ((p.Tq + 63) / 64) + LA_WAVES - 1) / LA_WAVES);
  else rb = reduce_blocks(riders.reduce);
  rb = (rb + 7) & ~7;
  if (p.Tq <= LS_MAX_ROWS && p.Tk <= LS_MAX_KEYS) {
    const int rt = p.Tq <= 32 ? 1 : 2, ksteps = p.Tk <= 64 ? 4 : 6, quads = (HZ_ELEMS / LS_COLS + 3) / 4;
    const unsigned wgs = (unsigned)std::min<long long>(ls_waves(ksteps, rt) * compute_units(), (long long)p.BH * quads);
#define LS_GO(KSTEPS, RT) { if (rb > 0) lin_short_kernel<KSTEPS, RT, true><<<wgs + rb, 256, 0, stream>>>(mbits, hz, p.Tq, p.Tk, p.BH, HZ, rb, riders); \
                            else lin_short_kernel<KSTEPS, RT, false><<<wgs, 256, 0, stream>>>(mbits, hz, p.Tq, p.Tk, p.BH, HZ, 0, riders); }
    if (ksteps == 4) { if (rt == 1) LS_GO(4, 1) else LS_GO(4, 2) }
    else { if (rt == 1) LS_GO(6, 1) else LS_GO(6, 2) }
#undef LS_GO
    return;
  }
  if (rb > 0) lin_accumulate_kernel<true><<<grid + rb, LA_WAVES * 64, 0, stream>>>(mbits, hz, p.Tq, p.Tk, groups, HZ, rb, p.BH, riders);
  else lin_accumulate_kernel<false><<<grid, LA_WAVES * 64, 0, stream>>>(mbits, hz, p.Tq, p.Tk, groups, HZ, 0, p.BH, riders);
}

}  // namespace sla
