// Key-block list of a work item, made by one wavefront without leaving registers and its own few words of
// LDS, while tile loads are in flight: table rows come through the scalar data path, whose waits do
// not touch those loads.
#ifndef BB_KEY_LIST_H_
#define BB_KEY_LIST_H_

#include "kernel_common.h"
#include "tile_ops.h"

namespace bb {

constexpr int kMaxListLen = 16;  // most key blocks of one item

// The lane number again, as a value the compiler cannot trace back.  Addresses and masks computed
// from it are then computed where they are used; computed from the known lane number they would
// be hoisted out of the item loop and carried through the pair loop, which has no register to
// spare (spilled, they come back one scratch load and one full memory wait at a time).
__device__ __forceinline__ int lane_again(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

// Key-block list of a non-global row without a padding mask, from the row of the pattern table
// that lanes 0 .. r-1 already hold in `rnd` (one entry per lane).  Same candidate order and
// rules as build_key_list_range: global blocks, window blocks, random blocks; a candidate is
// dropped if an earlier component already holds it.  Entries [lo, lo+len) go to klist.
__device__ __forceinline__ int finish_key_list_sparse(const Pattern& pat, int r, int j, int rnd, int lo,
                                                       int len, int lane, int* klist) {
  const int nb = pat.nb;
  const int ncand = pat.g + pat.w + r;  // <= 64 (checked by the caller)
  bool valid = false;
  int k = -1;
  const int t = lane - pat.g - pat.w;
  const int mine = __builtin_amdgcn_ds_bpermute((t < 0 ? 0 : t) * 4, rnd);  // entry t of the row, for the lanes that stand for it
  if (lane < pat.g) {
    k = pat.global_block(lane);
    valid = true;
  } else if (lane < pat.g + pat.w) {
    k = j - pat.half() + (lane - pat.g);
    valid = k >= 0 && k < nb && !pat.is_global(k);
  } else if (lane < ncand) {
    k = mine;
    valid = k >= 0 && k < nb && !pat.is_global(k) && !pat.in_window(j, k);
  }
  for (int u = 0; u < r; ++u) {
    const int ku = __builtin_amdgcn_readlane(rnd, u);
    if (u < t && ku == k) valid = false;
  }
  const uint64_t m = __ballot(valid);
  const int rank = mask_rank(m);
  if (valid && rank >= lo && rank < lo + len) klist[rank - lo] = k;
  int cnt = static_cast<int>(__popcll(m)) - lo;
  return cnt < 0 ? 0 : (cnt > len ? len : cnt);
}

// Up to four entries of a pattern-table row through the scalar data path: request and wait sit
// in one asm statement (the compiler sees the registers only once the values are in them), and
// the wait is on the scalar/LDS counter, which the tile loads in flight do not touch.
__device__ __forceinline__ void scalar_load4(const int32_t* row_, int o0, int o1, int o2, int o3, int (&e)[4]) {
  // wave uniform by construction; made so explicitly, or the operands may arrive in vector registers
  const int32_t* row = reinterpret_cast<const int32_t*>(uniform_ptr(reinterpret_cast<const char*>(row_)));
  o0 = __builtin_amdgcn_readfirstlane(o0);
  o1 = __builtin_amdgcn_readfirstlane(o1);
  o2 = __builtin_amdgcn_readfirstlane(o2);
  o3 = __builtin_amdgcn_readfirstlane(o3);
  asm volatile(
      "s_load_dword %0, %4, %5\n\t"
      "s_load_dword %1, %4, %6\n\t"
      "s_load_dword %2, %4, %7\n\t"
      "s_load_dword %3, %4, %8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&s"(e[0]), "=&s"(e[1]), "=&s"(e[2]), "=&s"(e[3])
      : "s"(row), "s"(o0 * 4), "s"(o1 * 4), "s"(o2 * 4), "s"(o3 * 4)
      : "memory");
}

// Does block j of batch entry bi hold a valid position?  The 64 mask bytes come through the scalar
// data path (request and wait in one statement, on the scalar counter): no vector memory wait, which
// would also wait for the tile loads in flight and for the stores of rows just written.
__device__ __forceinline__ bool block_any_valid_scalar(const uint8_t* kmask, int bi, int n, int j) {
  typedef __attribute__((ext_vector_type(16))) unsigned int u32x16;
  const char* ptr = uniform_ptr(reinterpret_cast<const char*>(kmask) + static_cast<size_t>(bi) * n + static_cast<size_t>(j) * kBlk);
  u32x16 v;
  asm volatile(
      "s_load_dwordx16 %0, %1, 0x0\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&s"(v)
      : "s"(ptr)
      : "memory");
  unsigned any = 0;
#pragma unroll
  for (int e = 0; e < 16; ++e) any |= v[e];
  return any != 0;
}

struct KeyList {
  int cnt;
  int entry;         // lane t holds entry t % 16
  unsigned partial;  // bit t: entry t has padded keys inside; its validity bits are in key_bits[t].
                     // Without key_bits: not 0 if any has
};

// Entries [lo, lo + len), len <= 16, of row j's list.  klist[16] and key_bits[16][2] (or NULL): this wave's, in LDS.
//
// Non-global rows: the list is made without a vector memory access.  A padding mask is then applied to
// the finished list, lane i looking at block i (one round trip to memory for the whole list) -- for rows
// of one slice, where dropping blocks afterwards cannot move a slice boundary.  Everything else takes the
// general builder.
template <bool kMask>
__device__ __forceinline__ KeyList item_key_list(const Pattern& pat, const int32_t* rand_idx, int r, const uint8_t* kmask,
                                                 int n, int bi, int h, int j, bool row_global, int lo, int len,
                                                 int lane, int* klist, uint32_t (*key_bits)[2]) {
  KeyList out;
  const bool masked = kMask && kmask;
  const bool fast_list = !row_global && rand_idx && r > 0 && pat.g + pat.w + r <= (masked ? kMaxListLen : 64);
  if (fast_list) {
    const int32_t* rrow = rand_idx + (static_cast<size_t>(h) * pat.nb + j) * r;
    int rnd = -1;
    for (int u0 = 0; u0 < r; u0 += 4) {
      int e[4];
      const int last = r - 1;
      scalar_load4(rrow, u0, u0 + 1 < last ? u0 + 1 : last, u0 + 2 < last ? u0 + 2 : last,
                   u0 + 3 < last ? u0 + 3 : last, e);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (lane == u0 + k && u0 + k < r) rnd = e[k];
    }
    // (without a mask there are registers for what is made of the lane number to stay in)
    out.cnt = finish_key_list_sparse(pat, r, j, rnd, lo, len, kMask ? lane : lane_id(), klist);
  } else {
    out.cnt = build_key_list_range(pat, rand_idx, r, kMask ? kmask : nullptr, n, bi, h, j, row_global, lo, len, kMask ? lane : lane_id(), klist);
  }
  // same wave wrote and reads the list: LDS keeps a wave's accesses in order, the compiler must too
  asm volatile("" ::: "memory");
  out.entry = klist[lane & (kMaxListLen - 1)];
  asm volatile("" ::: "memory");
  out.partial = 0;
  if (masked) {
    bool any_valid = false, any_padded = false;
    if (lane < out.cnt) block_mask_flags(kmask, bi, n, out.entry, any_valid, any_padded);
    const uint64_t m = __ballot(any_valid);
    const int place = fast_list ? mask_rank(m) : lane;
    const int kb = out.entry;
    if (fast_list) {
      // drop the blocks without a valid key (the general builder has done that already)
      if (any_valid) klist[place] = kb;
      out.cnt = static_cast<int>(__popcll(m));
    }
    const bool cut = any_valid && any_padded;
    if (!key_bits) {
      out.partial = __any(cut);
    } else if (__any(cut)) {
      if (cut) {
        uint32_t bits[2];
        block_key_bits(kmask, bi, n, kb, bits);
        key_bits[place][0] = bits[0];
        key_bits[place][1] = bits[1];
      }
      // entries are in lane order, so the flags of the kept lanes, closed up, are the flags of the list
      const uint64_t flags = __ballot(cut);
      if (fast_list) {
        unsigned closed = 0;
        uint64_t rest = m;
        for (int e = 0; rest; ++e, rest &= rest - 1)
          closed |= ((flags >> __builtin_ctzll(rest)) & 1) ? 1u << e : 0u;
        out.partial = closed;
      } else {
        out.partial = static_cast<unsigned>(flags);
      }
    }
    if (fast_list) {
      asm volatile("" ::: "memory");
      out.entry = klist[lane & (kMaxListLen - 1)];
      asm volatile("" ::: "memory");
    }
  }
  return out;
}

}  // namespace bb
#endif  // BB_KEY_LIST_H_
