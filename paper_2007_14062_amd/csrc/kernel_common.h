// Device-side helpers shared by the forward and backward kernels (gfx950 only).
#ifndef BB_KERNEL_COMMON_H_
#define BB_KERNEL_COMMON_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pattern_common.h"

namespace bb {

constexpr int kBlk = 64;      // block length b (App. E.1: 64 for every ITC model)
constexpr int kDim = 64;      // head width d
constexpr int kChunk = 8;     // list entries per slice of a global row / global key column
constexpr int kSparseChunk = 16;  // most key blocks per work item of a non-global row (the ITC base pattern has g+w+r = 8)
constexpr int kChunkGlobal = 8;  // key blocks per work item of a global row
constexpr int kChunkMax = kChunkGlobal > kSparseChunk ? kChunkGlobal : kSparseChunk;
constexpr int kXcd = 8;       // accelerator dies; workgroup id modulo 8 selects the die
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

#define BB_LDS __attribute__((address_space(3)))

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ float neg_inf() { return -__builtin_inff(); }

// v_exp_f32: 2^x, flushes tiny results to zero; arguments here are <= 0.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Value of x in the other 32-lane half of the wave, combined with max / add.
__device__ __forceinline__ float half_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Rank of this lane among the set bits of a wave-wide mask (number of set bits below it).
__device__ __forceinline__ int mask_rank(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
}

// Register-index -> row mapping of a 32x32 MFMA accumulator: element r of lane l
// sits in row 8*(r/4) + 4*(l/32) + r%4, column l%32.
__device__ __forceinline__ constexpr int acc_row(int r, int hf) { return 8 * (r >> 2) + 4 * hf + (r & 3); }

// Bank swizzle of a 64x64 bf16 tile kept in LDS with 128-byte rows: 16-byte chunk c of
// row `row` is stored at chunk position c ^ tile_swizzle(row).  LDS has 64 four-byte
// banks, so the row parity already selects a bank half and the swizzle uses row bits
// 1..3: bit 1 goes to position bit 2 (two rows of equal parity read by one transposing
// load then use different 64-byte halves), bits 2..3 to position bits 0..1 (the eight
// equal-parity rows read by one 16-lane pass of a 128-bit load get eight positions).
__device__ __forceinline__ int tile_swizzle(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

// Byte offset of 16-byte chunk c of row `row` in such a tile.
__device__ __forceinline__ int tile_off_bf16(int row, int chunk) {
  return row * 128 + ((chunk ^ tile_swizzle(row)) << 4);
}

// ds_read_b64_tr_b16: inside each group of 16 lanes, lane i passes the address of
// four 16-bit values (a piece of matrix row i/4, columns 4*(i%4)..+3) and gets back
// the four rows' values of column i -- a 4x16 block read transposed.
__device__ __forceinline__ s16x4 lds_read_tr16(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((BB_LDS s16x4*)(p));
}

constexpr int kF32Stride = 68;  // floats per row of an fp32 tile in LDS (64 + 4 padding)

// Decoded work item: which query block and which slice of its key-block list.
struct WorkItem {
  int bh;       // batch * H + head
  int j;        // query block
  int chunk;    // slice number: entries [chunk*len, (chunk+1)*len) of the row's key-block list
  int len;      // RowSplit::lg for a global row, RowSplit::ls otherwise
  int nchunks;  // slices this row is split into
  int slot;     // partial-result slot (valid when nchunks > 1)
  bool row_global;
};

// Launch geometry shared by forward and dQ: rows of global query blocks are split
// into cg slices, other rows into cs slices; global rows come first (longest first).
struct RowSplit {
  int lg, ls;         // key blocks per slice of a global / of a non-global row
  int cg, cs;         // slices per global / per non-global row
  int items_per_bh;   // g*cg + (nb-g)*cs
  int slots_per_bh;   // partial slots: (cg>1 ? g*cg : 0) + (cs>1 ? (nb-g)*cs : 0)
  int bh_rounds;      // ceil(B*H / 8)
};

// Longest key-block list of a non-global row.
inline int longest_sparse_list(int nb, int g, int w, int r) {
  const long long ub = static_cast<long long>(g) + w + r;
  return ub < nb ? static_cast<int>(ub) : nb;
}

// Block pairs of a launch, at most.
inline long long most_pairs(int BH, int nb, int g, int w, int r) {
  return BH * (static_cast<long long>(g) * nb + static_cast<long long>(nb - g) * longest_sparse_list(nb, g, w, r));
}

// Key blocks per slice of the fp32 kernels.  A block pair keeps a workgroup's matrix pipes busy for
// 2 .. 4 us there, so a launch that would have fewer than two 8-block slices per compute unit is cut finer,
// down to one pair per workgroup (n = 1024, 2 heads: forward 42 us with slices of 8, backward kernels
// 38 and 52; 13, 18 and 27 with slices of one).  0: use the standard slices.
// A length of 5 and more leaves a rest of one to three blocks of the usual list of 8, in a slice that costs
// nearly as much as a full one: 5 only where these slices still fit the chip at once (8 slices of n = 1792: forward
// and backward 37 and 115 us, 44 and 134 with 4), else 4 (8 of n = 2048: 55 and 166 us with 5, 44 and 147 with 4);
// from 6 on the standard ones (24 of n = 1024: 81 and 215 us with 7, 55 and 175 with 4, 47 and 162 with these).
inline int fine_slice_f32(int BH, int nb, int g, int w, int r) {
  const int sparse = longest_sparse_list(nb, g, w, r);
  const long long len = (most_pairs(BH, nb, g, w, r) + 511) / 512;
  if (len > 5) return 0;
  if (len == 5)
    return static_cast<long long>(BH) * (static_cast<long long>(g) * ((nb + 4) / 5) + static_cast<long long>(nb - g) * ((sparse + 4) / 5)) <= 512 ? 5 : 4;
  return static_cast<int>(len < 1 ? 1 : len);
}

// len: key blocks per slice of every row; 0: global_len / kSparseChunk.
inline RowSplit make_row_split(int BH, int nb, int g, int w, int r, int len = 0, int global_len = kChunkGlobal) {
  RowSplit s;
  const int sparse_ub = longest_sparse_list(nb, g, w, r);
  s.lg = len > 0 ? len : global_len;
  s.ls = len > 0 ? len : kSparseChunk;
  s.cg = (nb + s.lg - 1) / s.lg;
  s.cs = (sparse_ub + s.ls - 1) / s.ls;
  if (s.cs < 1) s.cs = 1;
  s.items_per_bh = g * s.cg + (nb - g) * s.cs;
  s.slots_per_bh = (s.cg > 1 ? g * s.cg : 0) + (s.cs > 1 ? (nb - g) * s.cs : 0);
  s.bh_rounds = (BH + kXcd - 1) / kXcd;
  return s;
}

// Hardware hands consecutive workgroup ids to the 8 dies round robin, so id % 8 picks the die.  Die x
// gets the (batch, head) slices x, x + 8, ... whole, so that a slice's K and V (1 MB at n = 4096) stay in
// its L2 and the sequences of a padded batch are spread over the dies; the items of the last B * H mod 8
// slices are cut into eight equal runs: whole slices would leave six dies idle at B * H = 2 (fp32
// forward at n = 1024, one pair per item: 25 us against 13) and give four of them twice the work of
// the others at 12 (bf16 dQ and dK/dV kernels at n = 1088: 16 and 21 us against 13 and 18).
struct DieItems {
  unsigned rounds;   // whole slices per die
  unsigned per_bh;   // items per slice
  unsigned total;    // items of the slices left over
  unsigned run;      // of these per die
  __host__ __device__ DieItems(int BH, int items_per_bh) {
    rounds = BH / kXcd;
    per_bh = items_per_bh;
    total = (BH % kXcd) * per_bh;
    run = (total + kXcd - 1) / kXcd;
  }
  unsigned grid() const { return kXcd * (rounds * per_bh + run); }
  // workgroup -> (slice, item); false: none.  interleaved: the items of up to `interleaved` of the die's
  // slices alternate (for items that come longest first), instead of slice after slice.
  __device__ __forceinline__ bool decode(unsigned wg, int* bh, int* item, unsigned interleaved = 1) const {
    const unsigned xcd = wg % kXcd, u = wg / kXcd;
    if (u < rounds * per_bh) {
      const unsigned groups = (rounds + interleaved - 1) / interleaved, size = (rounds + groups - 1) / groups;
      const unsigned base = u / per_bh / size * size, n = rounds - base < size ? rounds - base : size;
      const unsigned v = u - base * per_bh;
      *bh = static_cast<int>((base + v % n) * kXcd + xcd);
      *item = static_cast<int>(v / n);
      return true;
    }
    const unsigned t = xcd * run + (u - rounds * per_bh);
    *bh = static_cast<int>(rounds * kXcd + t / per_bh);
    *item = static_cast<int>(t % per_bh);
    return u < rounds * per_bh + run && t < total;
  }
};

// Workgroup id -> work item.
__device__ __forceinline__ bool decode_item(const RowSplit& s, const Pattern& pat, int BH,
                                            unsigned wg, WorkItem* it) {
  int item;
  if (!DieItems(BH, s.items_per_bh).decode(wg, &it->bh, &item)) return false;
  const int nglob = pat.g * s.cg;
  if (item < nglob) {
    it->row_global = true;
    it->len = s.lg;
    it->j = pat.global_block(item / s.cg);
    it->chunk = item % s.cg;
    it->nchunks = s.cg;
    it->slot = it->bh * s.slots_per_bh + item;
  } else {
    const int t = item - nglob;
    it->row_global = false;
    it->len = s.ls;
    it->j = pat.sparse_block(t / s.cs);
    it->chunk = t % s.cs;
    it->nchunks = s.cs;
    it->slot = it->bh * s.slots_per_bh + (s.cg > 1 ? nglob : 0) + t;
  }
  return true;
}

// Does key block k of batch bi hold at least one valid key?  (64 mask bytes)
__device__ __forceinline__ bool block_has_valid_key(const uint8_t* kmask, int bi, int n, int k) {
  const u32x4* p = reinterpret_cast<const u32x4*>(kmask + static_cast<size_t>(bi) * n + k * kBlk);
  unsigned any = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    u32x4 v = p[i];
    any |= v[0] | v[1] | v[2] | v[3];
  }
  return any != 0;
}

// The 64 mask bytes of key block k of batch bi (a byte is a flag): is any key valid, is any padded?
__device__ __forceinline__ void block_mask_flags(const uint8_t* kmask, int bi, int n, int k, bool& any_valid,
                                                 bool& any_padded) {
  const u32x4* p = reinterpret_cast<const u32x4*>(kmask + static_cast<size_t>(bi) * n + k * kBlk);
  unsigned any = 0, zero_byte = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u32x4 v = p[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      any |= v[e];
      zero_byte |= (v[e] - 0x01010101u) & ~v[e] & 0x80808080u;  // some byte of v[e] is 0
    }
  }
  any_valid = any != 0;
  any_padded = zero_byte != 0;
}

// The same 64 bytes as bits (bit t of bits[0] / bits[1]: key t / 32 + t of the block is valid).
__device__ __forceinline__ void block_key_bits(const uint8_t* kmask, int bi, int n, int k, uint32_t (&bits)[2]) {
  const u32x4* p = reinterpret_cast<const u32x4*>(kmask + static_cast<size_t>(bi) * n + k * kBlk);
  bits[0] = bits[1] = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u32x4 v = p[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t set = ((((v[e] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v[e]) >> 7) & 0x01010101u;  // byte != 0
      // bits 0, 8, 16, 24 -> bits 24 .. 27 (no two products meet)
      bits[i >> 1] |= ((set * 0x01020408u) >> 24 & 15u) << ((i & 1) * 16 + e * 4);
    }
  }
}

// Key blocks attended by query block j of head h (App. D items 1-3 as a set
// union, minus blocks without a valid key), slice `chunk` (see WorkItem) of the
// ascending-by-candidate list: entries [lo, lo+len).  Every lane of the calling wave takes
// part; the slice is written to klist[0..count) and the count returned (wave uniform).
// Candidate order: global blocks, window blocks, random blocks; a candidate is
// dropped if an earlier component already holds it.
__device__ __forceinline__ int build_key_list_range(const Pattern& pat, const int32_t* rand_idx, int r,
                                                    const uint8_t* kmask, int n, int bi, int h, int j,
                                                    bool row_global, int lo, int len, int lane, int* klist) {
  const int nb = pat.nb;
  const int ncand = row_global ? nb : pat.g + pat.w + r;
  const int hi = lo + len;
  const int32_t* rrow = rand_idx ? rand_idx + (static_cast<size_t>(h) * nb + j) * r : nullptr;
  int base = 0;
  for (int c0 = 0; c0 < ncand && base < hi; c0 += 64) {
    const int ci = c0 + lane;
    bool valid = false;
    int k = -1;
    if (ci < ncand) {
      if (row_global) {
        k = ci;
        valid = true;
      } else if (ci < pat.g) {
        k = pat.global_block(ci);
        valid = true;
      } else if (ci < pat.g + pat.w) {
        k = j - pat.half() + (ci - pat.g);
        valid = k >= 0 && k < nb && !pat.is_global(k);
      } else if (rrow) {
        const int t = ci - pat.g - pat.w;
        k = rrow[t];
        valid = k >= 0 && k < nb && !pat.is_global(k) && !pat.in_window(j, k);
        for (int u = 0; u < t && valid; ++u) valid = rrow[u] != k;
      }
      if (valid && kmask) valid = block_has_valid_key(kmask, bi, n, k);
    }
    const uint64_t m = __ballot(valid);
    const int rank = base + mask_rank(m);
    if (valid && rank >= lo && rank < hi) klist[rank - lo] = k;
    base += __popcll(m);
  }
  int cnt = base - lo;
  cnt = cnt < 0 ? 0 : (cnt > len ? len : cnt);
  return cnt;
}

// The same for a work item's slice.
__device__ __forceinline__ int build_key_list(const Pattern& pat, const int32_t* rand_idx, int r,
                                              const uint8_t* kmask, int n, int bi, int h, const WorkItem& it,
                                              int* klist) {
  return build_key_list_range(pat, rand_idx, r, kmask, n, bi, h, it.j, it.row_global, it.chunk * it.len, it.len, lane_id(), klist);
}

// 64-bit validity mask of the keys of block k (bit t = key k*64+t is valid).
__device__ __forceinline__ uint64_t key_valid_bits(const uint8_t* kmask, int bi, int n, int k) {
  const uint8_t v = kmask[static_cast<size_t>(bi) * n + k * kBlk + lane_id()];
  return __ballot(v != 0);
}

}  // namespace bb
#endif  // BB_KERNEL_COMMON_H_
