// Device code of the block classification that more than one launch runs: the selection of one row's blocks, and the
// statistics that have to be joined over all blocks of a slice.
#pragma once
#include "common.h"

namespace sla {

// select_row: one WAVEFRONT per (b,h,i) row; the row's scores (score(j), j < Tk) live in registers (KPL per lane,
// block j = lane + 64 m in register m) as order-preserving 32-bit keys.  The n_c-th and the
// (n_c+n_m)-th largest keys are found exactly, bit by bit from the top: a bit of the threshold
// is set when at least `rank` keys are >= the candidate with that bit set.  The counts come
// from wave-wide compares (one vector compare per register, the population count and the sum
// on the scalar unit), so there is no shared-memory traffic and no atomic.  Blocks whose key
// equals a threshold key are ranked by ascending j with ballots, so equal scores rank by
// ascending block index and the result is exact and deterministic.  Outputs: the int8 mask
// row, the ascending critical list, and the marginal ballots as words of the bit matrix the
// accumulation kernel reads (see lin_accumulate).
__device__ __forceinline__ uint32_t order_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

struct ScoresOf {
  const float* row;
  __device__ __forceinline__ float operator()(int j) const { return row[j]; }
};
template <int KPL, class Score>
__device__ __forceinline__ void select_row(const SelectArgs& S, unsigned row_, Score score) {
  const size_t row = row_;
  const int Tq = S.Tq, Tk = S.Tk, n_c = S.n_c, n_m = S.n_m;
  const int lane = threadIdx.x & 63;
  const unsigned long long lt = (1ull << lane) - 1ull;
  uint32_t key[KPL];
#pragma unroll
  for (int m = 0; m < KPL; ++m) {
    const int j = lane + 64 * m;
    key[m] = j < Tk ? order_bits(score(j)) : 0u;
  }
  // Subtract the row minimum and shift out the common leading zeros: order and ties are
  // unchanged, padding (key 0) ties with the minimum, and the search below only has to visit
  // the bits in which the keys can differ.
  int low;
  {
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int m = 0; m < KPL; ++m)
      if (lane + 64 * m < Tk) {
        kmin = min(kmin, key[m]);
        kmax = max(kmax, key[m]);
      }
    kmin = __builtin_amdgcn_readfirstlane(rows_reduce(row_reduce(kmin, OpMin{}), OpMin{}));
    kmax = __builtin_amdgcn_readfirstlane(rows_reduce(row_reduce(kmax, OpMax{}), OpMax{}));
    const uint32_t span = kmax - kmin;
    const int lz = span ? __builtin_clz(span) : 0;
    low = span ? lz : 32;  // all keys equal: nothing to search
#pragma unroll
    for (int m = 0; m < KPL; ++m) key[m] = (lane + 64 * m < Tk) ? ((key[m] - kmin) << lz) : 0u;  // padding ties with the minimum: never above a threshold
  }
  // k1 / k2: the n_c-th / (n_c+n_m)-th largest key; t1 / t2: how many of the keys equal to
  // it belong to the top n_c / n_c+n_m (>= 1).  Bits below `low` are zero in every key.
  // A threshold's search stops early once exactly the wanted number of keys reaches the
  // candidate c: the set is then {key >= c}, which the code below takes as "key > c - 1" with
  // no ties to rank (with ~1000 distinct keys that happens after about log2(Tk) + 2 bits).
  uint32_t k1 = 0, k2 = 0;
  const int rank2 = n_c + n_m;
  bool open1 = true, open2 = n_m > 0;
  for (int bit = 31; bit >= low && (open1 || open2); --bit) {
    const uint32_t c1 = k1 | (1u << bit), c2 = k2 | (1u << bit);
    int n1 = 0, n2 = 0;
#pragma unroll
    for (int m = 0; m < KPL; ++m) {  // (padding keys are 0 and never reach a candidate)
      if (open1) n1 += __popcll(__ballot(key[m] >= c1));
      if (open2) n2 += __popcll(__ballot(key[m] >= c2));
    }
    if (open1) {
      if (n1 == n_c) { k1 = c1 - 1u; open1 = false; }
      else if (n1 > n_c) k1 = c1;
    }
    if (open2) {
      if (n2 == rank2) { k2 = c2 - 1u; open2 = false; }
      else if (n2 > rank2) k2 = c2;
    }
  }
  int t1 = n_c, t2 = rank2;
#pragma unroll
  for (int m = 0; m < KPL; ++m) {
    t1 -= __popcll(__ballot(key[m] > k1));
    if (n_m > 0) t2 -= __popcll(__ballot(key[m] > k2));
  }

  const int bh = (int)(row_ / (unsigned)Tq), i = (int)(row_ - (unsigned)bh * (unsigned)Tq);
  const int KT = (Tk + 31) / 32, TqP = (Tq + 383) / 384 * 384 + 128;  // layout of the marginal bit matrix (see lin_accumulate)
  int eq1 = 0, eq2 = 0, nc = 0, nm = 0;  // running counts in ascending-j order
#pragma unroll
  for (int m = 0; m < KPL; ++m) {
    const int j = lane + 64 * m;
    if (64 * m >= Tk) break;
    const bool valid = j < Tk;
    const bool e1 = valid && key[m] == k1, e2 = valid && n_m > 0 && key[m] == k2;
    const unsigned long long b1 = __ballot(e1), b2 = __ballot(e2);
    const int r1 = eq1 + __popcll(b1 & lt), r2 = eq2 + __popcll(b2 & lt);
    eq1 += __popcll(b1);
    eq2 += __popcll(b2);
    const bool is_c = valid && (key[m] > k1 || (e1 && r1 < t1));
    const bool is_m = valid && !is_c && n_m > 0 && (key[m] > k2 || (e2 && r2 < t2));
    if (S.mask && valid) S.mask[row * Tk + j] = is_c ? 1 : (is_m ? 0 : -1);
    const unsigned long long bc = __ballot(is_c), bm = __ballot(is_m);
    if (S.crit && is_c) S.crit[row * n_c + nc + __popcll(bc & lt)] = j;
    if (S.marg && is_m) S.marg[row * n_m + nm + __popcll(bm & lt)] = j;
    nc += __popcll(bc);
    nm += __popcll(bm);
    if (S.mbits && lane < 2) {  // the marginal ballot of these 64 key blocks = two words of the bit matrix
      const int kt = 2 * m + lane;
      if (kt < KT) S.mbits[((size_t)bh * KT + kt) * TqP + i] = (uint32_t)(bm >> (32 * lane));
    }
  }
}

// The mean of K is the sum of MEAN_RUNS interleaved partial sums over the key blocks (j, j + 64, ...; cnt_j tokens times
// the block's mean, one fma each), added in ascending order: the INT8 codes of K hang on its last bit, so the order of
// summation is part of the result.
constexpr int MEAN_RUNS = 64;

}  // namespace sla
