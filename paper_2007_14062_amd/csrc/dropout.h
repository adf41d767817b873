// Attention dropout: the keep mask as a function of (seed, batch*H + head, query, key).
//
// The paper names only the rate (App. E.1: "attention dropout 0.1").  Here an attended
// probability P_ij is kept with probability 1 - p and the kept ones are scaled by 1 / (1 - p);
// LSE stays that of the undropped softmax.  The mask must be the same in the forward and in both
// backward kernels, whatever their tiling, so it is computed from the element's coordinates by a
// counter-based generator on 32-bit integers (arithmetic modulo 2^32):
//   mix(x):  x ^= x >> 16; x *= 0x7feb352d; x ^= x >> 15; x *= 0x846ca68b; x ^= x >> 16
//   row key  rk(i)   = mix(seed_lo ^ mix(seed_hi ^ (bh * n + i)))
//   word     w(i, j) = mix(rk(i) ^ ((j >> 1) * 0x9E3779B9))      -- one word per pair of keys
//   number   u(i, j) = bits 0..14 of w for even j, bits 16..30 for odd j
//   keep     u(i, j) >= T,  T = round(p * 32768)
// so the rate realised is T / 32768 and the scale 32768 / (32768 - T).  A row key costs two
// mixes per (query, work item); a word serves the two keys that share a packed bf16 register in
// the kernels whose lanes own a query.
#ifndef BB_DROPOUT_H_
#define BB_DROPOUT_H_

#include <stdint.h>

#include "pattern_common.h"

namespace bb {

struct Dropout {
  uint32_t thr;      // T; 0 = no dropout
  uint32_t seed_lo, seed_hi;
  float rs;          // 32768 / (32768 - T); 1 without dropout
};

BB_HD uint32_t drop_mix(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

// rowid = (batch*H + head) * n + query, as a 32-bit number
BB_HD uint32_t drop_row_key(const Dropout& dr, uint32_t rowid) {
  return drop_mix(dr.seed_lo ^ drop_mix(dr.seed_hi ^ rowid));
}

// the word of keys 2*pair and 2*pair + 1
BB_HD uint32_t drop_word(uint32_t rk, uint32_t pair) { return drop_mix(rk ^ (pair * 0x9E3779B9u)); }

BB_HD bool drop_keep_even(uint32_t w, uint32_t thr) { return (w & 0x7fffu) >= thr; }
BB_HD bool drop_keep_odd(uint32_t w, uint32_t thr) { return ((w >> 16) & 0x7fffu) >= thr; }

BB_HD bool drop_keep(const Dropout& dr, uint32_t rowid, uint32_t key) {
  const uint32_t w = drop_word(drop_row_key(dr, rowid), key >> 1);
  return (key & 1u) ? drop_keep_odd(w, dr.thr) : drop_keep_even(w, dr.thr);
}

#if defined(__HIPCC__)
// The same in the form the bf16 kernels use, with fewer instructions for a word:
//   * the first step of mix is linear over xor, so it is done once for a row key and once for a pair of keys
//     (drop_first) and not for every (row, pair); the pairs' side comes from a small table in LDS;
//   * with twice the second factor the numbers end up doubled, in bits 1..15 and 17..31 of one word, each above a
//     bit that does not matter: 2 u + (0 or 1) >= 2 T if and only if u >= T.  That saves masking them.
// Words are what bounds the kernels under dropout (vector port; 32 of them a block pair and wave): 8 instructions each and 3
// to apply one, where it were 9 and 3 and the two of the argument.  Step of 48 slices of n = 3072, padded: 150 -> 141 us.
constexpr uint32_t kDropPairStep = 0x9E3779B9u;
__device__ __forceinline__ uint32_t drop_first(uint32_t x) { return x ^ (x >> 16); }
// x = drop_first(row key) ^ drop_first(pair * kDropPairStep): low half even key, upper half odd key
__device__ __forceinline__ uint32_t drop_doubled(uint32_t x) {
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 2u * 0x846ca68bu;
  // (x ^ x >> 16 in one instruction, whatever is made of the halves)
  asm("v_xor_b32_sdwa %0, %0, %0 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "+v"(x));
  return x;
}
__device__ __forceinline__ bool drop_keep_low(uint32_t doubled, uint32_t thr) { return static_cast<uint16_t>(doubled) >= static_cast<uint16_t>(2u * thr); }
__device__ __forceinline__ bool drop_keep_high(uint32_t doubled, uint32_t thr) { return doubled >= thr << 17; }
// Both keys at once: 1 in each half that is kept, else 0 (a packed subtraction that stops at 0, and a minimum; written
// out, because the compiler knows them for comparisons and makes six instructions of those).
__device__ __forceinline__ uint32_t drop_pair_threshold(const Dropout& dr) { return (2u * dr.thr - 1u) * 0x10001u; }
__device__ __forceinline__ uint32_t drop_keep_pair(uint32_t doubled, uint32_t threshold) {
  uint32_t keep;
  asm("v_pk_sub_u16 %0, %1, %2 clamp\n\tv_pk_min_u16 %0, %0, 1 op_sel_hi:[1,0]" : "=v"(keep) : "v"(doubled), "s"(threshold));
  return keep;
}
// Two packed 16-bit values, each of them or 0.
__device__ __forceinline__ uint32_t drop_apply(uint32_t values, uint32_t keep) {
  asm("v_pk_mul_lo_u16 %0, %0, %1" : "+v"(values) : "v"(keep));
  return values;
}

// Kernels whose lanes own a query: drop_first of the 32 key pairs of a block, left in LDS by the wave that needs them.  A lane of
// half hf reads those of a unit of 32 keys together: element m belongs to accumulator registers 2 m, 2 m + 1.
__device__ __forceinline__ void drop_key_words(uint32_t* table, uint32_t kblock, int lane) {
  const uint32_t i = static_cast<uint32_t>(lane) & 31u;  // (both halves of the wave write the same)
  table[(i & 17u) | ((i & 2u) << 2) | ((i & 12u) >> 1)] = drop_first((kblock * 32u + i) * kDropPairStep);
  asm volatile("" ::: "memory");  // read by the same wave: LDS keeps the order, the compiler must too
}
__device__ __forceinline__ const uint32_t* drop_unit_words(const uint32_t* table, int t, int hf) { return table + t * 16 + hf * 8; }
#endif

// Host: rate and seed -> parameters.  False if p is not in [0, 1) or rounds to 1.
inline bool make_dropout(float p, uint64_t seed, Dropout* out) {
  if (!(p >= 0.f) || !(p < 1.f)) return false;
  const uint32_t t = static_cast<uint32_t>(static_cast<double>(p) * 32768.0 + 0.5);
  if (t >= 32768u) return false;
  out->thr = t;
  out->seed_lo = static_cast<uint32_t>(seed);
  out->seed_hi = static_cast<uint32_t>(seed >> 32);
  out->rs = static_cast<float>(32768.0 / (32768.0 - static_cast<double>(t)));
  return true;
}

}  // namespace bb
#endif  // BB_DROPOUT_H_
