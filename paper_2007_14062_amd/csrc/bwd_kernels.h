// Launch interface of the backward kernels (internal to the library).
#ifndef BB_BWD_KERNELS_H_
#define BB_BWD_KERNELS_H_

#include "dropout.h"
#include "kernel_common.h"

namespace bb {

constexpr int kMaxBwdBlocks = 256;  // longest query-block list a key block can have (LDS list): n <= 16 384,
                                    // the longest sequence the backward is verified on in full

// dK/dV launch geometry: the query-block list of a global key block is cut into cg slices, that of
// another one into cs slices; slice u of c takes entries u, u + c, ... of the list.
struct KeySplit {
  int cg, cs;
  int items_per_bh;  // g*cg + (nb-g)*cs
  int slots_per_bh;  // partial slots: (cg>1 ? g*cg : 0) + (cs>1 ? (nb-g)*cs : 0)
};

// len: list entries per slice of every key block (of an average list where its length is not known);
// 0: global_len for a global key block, one slice for the others.
inline KeySplit make_key_split(int nb, int g, int w, int r, int len = 0, int global_len = kChunk) {
  KeySplit s;
  s.cg = (nb + (len > 0 ? len : global_len) - 1) / (len > 0 ? len : global_len);
  s.cs = len > 0 ? (longest_sparse_list(nb, g, w, r) + len - 1) / len : 1;
  if (s.cs < 1) s.cs = 1;
  s.items_per_bh = g * s.cg + (nb - g) * s.cs;
  s.slots_per_bh = (s.cg > 1 ? g * s.cg : 0) + (s.cs > 1 ? (nb - g) * s.cs : 0);
  return s;
}

// Small bf16 launches: a workgroup per query block (dQ) and per key block (dK/dV) that deals out the block's
// list to four waves or pairs of waves.  Otherwise most of the chip is idle behind lists of eight pairs in
// series.
constexpr int kRowWaves = 4;
// Entries per wave (pair of waves) of a global block's list: all of it in one workgroup up to 8 each, which
// saves the reduction launch; longer lists in several workgroups of 4 each, so that they end with the others (2 heads,
// n = 4096: 25 us, with 16 each 43).
inline int by_row_share(int nb) {
  const int quarter = (nb + kRowWaves - 1) / kRowWaves;
  return quarter <= 8 ? quarter : 4;
}
// dQ items then; a non-global row whole.
inline RowSplit make_row_split_by_row(int BH, int nb, int g, int w, int r) {
  RowSplit s = make_row_split(BH, nb, g, w, r);
  const int sparse = (longest_sparse_list(nb, g, w, r) + kRowWaves - 1) / kRowWaves;
  s.lg = kRowWaves * by_row_share(nb);
  s.ls = kRowWaves * (sparse > 1 ? sparse : 1);
  s.cg = (nb + s.lg - 1) / s.lg;
  s.cs = 1;
  s.items_per_bh = g * s.cg + nb - g;
  s.slots_per_bh = s.cg > 1 ? g * s.cg : 0;
  return s;
}
// dK/dV items.
inline KeySplit make_key_split_by_row(int nb, int g) {
  KeySplit s;
  s.cg = (nb + kRowWaves * by_row_share(nb) - 1) / (kRowWaves * by_row_share(nb));
  s.cs = 1;
  s.items_per_bh = g * s.cg + nb - g;
  s.slots_per_bh = s.cg > 1 ? g * s.cg : 0;
  return s;
}
// Where that wins: up to a dK/dV workgroup per compute unit.  12 heads, n = 512 / 1088 / 1344, whole backward:
// 25.5 -> 18.1, 32.5 -> 24.7, 32.9 -> 27.5 us; 2 heads, n = 4096: 32.0 -> 24.9.  Past that some units have two, one
// after the other: 4 slices of n = 4096 (280 workgroups) 34.0 -> 34.2, one of n = 16384 (286) 37.4 -> 39.7.
inline bool bwd_by_row(int BH, int nb, int g, int w, int r) {
  return static_cast<long long>(BH) * make_key_split_by_row(nb, g).items_per_bh <= 256 &&
         longest_sparse_list(nb, g, w, r) <= kRowWaves * kChunkMax;
}

// Between the small launches and those that put two dQ items on every SIMD: two waves per item, which deal out its
// list (or its slice of up to 16 blocks) in halves.  From 384 items, where single waves would leave most SIMDs empty, up to
// 1024, where two per item fill them.  Whole backward, one wave / two: 24 slices of n = 1024 (432 items) 36.7 / 35.4 us,
// 72 of n = 640 (864) 48 / 43 and under dropout 70 / 59, 36 of n = 1536 (1008) 54 / 48.  Past 1024 items 58 / 58 (48
// of n = 1280) and 62 / 66 (72 of n = 1024); below 384 as often slower as faster (12 of n = 1536, 336 items: 34.2 / 35.4).
inline bool dq_two_waves(int BH, const RowSplit& s) {
  const long long items = static_cast<long long>(BH) * s.items_per_bh;
  return items >= 384 && items <= 1024;
}

// The same for dK/dV: two pairs of waves per item up to 512 items, all resident at once (four waves each). Past that
// they queue.  Forward and backward in us, one pair / two: 24 slices of n = 1024 (432 items) 50.8 / 49.9 and under dropout
// 84 / 78, 12 of n = 2048 (456) 53.1 / 50.7, with w = 7 62 / 58, padded 56.5 / 53.0, under dropout 90 / 81, 48 of n = 512 (384)
// 42.0 / 39.8, 4 of n = 4096 (312) 50.2 / 48.6; 8 of n = 2048 (304) and 16 of n = 1024 (288) the same.  Past 512 items:
// 12 of n = 2048 with four global blocks (528) 63.3 / 67.1, 24 of n = 1536 (672) 57.3 / 58.5, 12 of n = 4096 (936) 67 / 72, 24 (1872) 101.5 / 111.
// Short lists leave the second pair one entry or none, and only gain where it lets a second workgroup onto a unit: one block
// 15.8 / 16.4 (384 slices), 96 of n = 192 (288 items) 17.9 / 19.0, 72 of n = 256 (288) 19.2 / 20.1, 48 of n = 384 (288) 23.4 / 24.2,
// but 64 of n = 384 (384) 26.7 / 25.6 and under dropout 40 / 35, 96 of n = 256 (384) 21.9 / 21.0 and 31 / 28.
inline bool dkv_two_teams(int BH, int nb, const KeySplit& s) {
  const long long items = static_cast<long long>(BH) * s.items_per_bh;
  return items <= 512 && nb > 1 && (nb > 6 || items > 288);
}

// Slices of a die whose items alternate in the dK/dV kernels, in groups as equal as they come: as many as have their Q and
// dO (256 n bytes each) in an L2 together.  With the longest lists of all of them first the bf16 kernel ends sooner (24
// slices, n = 4096: 43 -> 42 us; 48 padded ones, n = 3072, dropout: 64 -> 60), but two slices of n = 16384 alternating
// miss the L2 (104 -> 111).
__host__ __device__ inline int key_slices_together(int n) { return n < 16384 ? 16384 / n : 1; }

// Large bf16 launches: slices of global blocks longer than the standard 8, where the launch is long enough that
// they still end with the others (the longest items start first).  Every slice costs 16 KB (dQ) or 32 KB (dK/dV) written
// and read again by the reduction.  The lines lie by the pairs each resident workgroup gets on average: 1024 of the dK/dV
// kernel, 2048 of the dQ kernel.  Forward and backward in us, dK/dV slices of 8 / 16 / 24 / 32:
//   40 pairs: 16 slices of n = 16384   263 / 260 / 257 / 255; 32 of n = 8192  257 / 255 / 251 / 247
//   29: 48 of n = 4096  191 / 187 / 184 / 187; 96 of n = 2048  191 / 186 / 184 / 187; 64 of n = 3072  193 / 188 / 187 / 187
//   14..20: 16 of n = 8192  134 / 133 / 130 / 132; 24 of n = 4096  100.5 / 99.8 / 99.4 / 101.7; 64 of n = 1536  98.5 / 98.6 / 95.5 / 95.4
//   9..10: 8 of n = 8192  79 / 80 / 80 / 87; 20 of n = 3072  82 / 81 / 89 / 90
// Where slices of a launch are left over and cut into runs (DieItems), longer items make the runs uneven: 12 of n = 12288
// (22 pairs, slices of 8 / 12 / 16 / 24) 160 / 159 / 158 / 164, 36 of n = 2560 (14) 99.5 / 99.6 / 100.5 / 103.3.  Under a mask
// lists are shorter than counted: 48 padded ones of n = 3072, dropout (8 / 16 / 24) 139.9 / 138.8 / 144.5.
// Under dropout, where a pair takes longest, the last of the groups of slices that are worked on together (key_slices_together)
// may be smaller than the others, and its long items start late: whole backward, slices of 8 / 12 / 16 / 24, 24 of n = 6464 (groups
// of 2 and 1 on a die) 150 / 148 / 149 / 166, 24 of n = 5760 144 / 143 / 145 / 151, 40 of n = 4608 (3 and 2) 182 / 177 / 179 / 185; with equal
// groups 48 of n = 4096 (3 and 3) 196 / 192 / 192 / 192.
inline int dkv_global_slice(int BH, int nb, int g, int w, int r, bool masked, bool drop) {
  const long long each = most_pairs(BH, nb, g, w, r) / 1024;
  if (each < 14) return kChunk;
  if (BH % kXcd != 0) return 12;
  if (masked) return 16;
  const int slices = BH / kXcd, together = key_slices_together(nb * kBlk), groups = (slices + together - 1) / together;
  if (drop && slices % groups != 0) return 12;
  return each < 32 ? 24 : 32;
}
// dQ slices of 8 / 16 (the most a wave lists): 20 pairs: 16 slices of n = 16384  255 / 248, 32 of n = 8192  247 / 246; 15: 48 of
// n = 4096  187 / 188, 64 of n = 3072  187 / 189; 7: 24 of n = 4096  102 / 106.
inline int dq_global_slice(int BH, int nb, int g, int w, int r, bool masked) {
  return !masked && most_pairs(BH, nb, g, w, r) / 2048 >= 18 ? 2 * kChunkGlobal : kChunkGlobal;
}

constexpr int kSetWords = kMaxBwdBlocks / 32;

struct BwdParams {
  const void* Q;
  const void* K;
  const void* V;
  const void* O;
  const void* dO;
  const float* LSE;
  float* dQ;
  float* dK;
  float* dV;
  const int32_t* rand_idx;
  const uint8_t* kmask;
  // written by the dQ kernel for the dK/dV kernel
  float* Dvec;     // [B*H*n]  bf16: -D_i, D_i = sum_c dO_ic O_ic; fp32: D_i
  float* Lvec;     // [B*H*n]  LSE_i * log2(e), +inf for rows without a valid key
  int* key_order;  // bf16: [H][nb] non-global key blocks by falling length of their query-block lists
  uint32_t* query_sets;  // bf16: [H][nb][kSetWords] query blocks that attend a non-global key block, as bits
  unsigned inverse_wgs;  // bf16: workgroups of the dQ launch that make these (a multiple of the dies)
  float* part_dq;  // [slots][64][64] partial dQ of split rows (slots as in the forward)
  float* part_dk;  // [slots][64][64] partial dK of split key blocks (slots: see KeySplit)
  float* part_dv;  // same for dV
  int B, H, BH, n, nb, g, w, r, global_mode;
  float c;      // scale * log2(e)
  float scale;
  int by_row;      // bf16: a workgroup per block (bwd_by_row)
  int dq_waves;    // bf16: waves of a dQ item: kRowWaves if by_row, else 1 or 2 (dq_two_waves)
  int dkv_teams;   // bf16: pairs of waves of a dK/dV item: kRowWaves if by_row, else 1 or 2 (dkv_two_teams)
  RowSplit split;  // query-row decomposition (dQ kernel), as in the forward
  KeySplit kv;     // key-block decomposition (dK/dV kernel)
  Dropout drop;    // attention dropout of the forward these gradients belong to (thr == 0: none)
  int skip_q;      // query blocks without a valid position (in kmask) were not computed: no gradient through them
};

// One item of the dK/dV kernels.
struct KeyItem {
  int bh, k;
  int chunk, nchunks, slot;
  bool key_global;
};

// Workgroup id -> item (see decode_item).  False: no such item.
__device__ __forceinline__ bool decode_key_item(const BwdParams& p, const Pattern& pat, unsigned wg, KeyItem* it) {
  int item;
  if (!DieItems(p.BH, p.kv.items_per_bh).decode(wg, &it->bh, &item, key_slices_together(p.n))) return false;
  const int nglob = p.g * p.kv.cg;
  it->key_global = item < nglob;
  if (it->key_global) {
    it->k = pat.global_block(item / p.kv.cg);
    it->chunk = item % p.kv.cg;
    it->nchunks = p.kv.cg;
    it->slot = it->bh * p.kv.slots_per_bh + item;
  } else {
    const int t = item - nglob;
    it->k = pat.sparse_block(t / p.kv.cs);
    it->chunk = t % p.kv.cs;
    it->nchunks = p.kv.cs;
    it->slot = it->bh * p.kv.slots_per_bh + (p.kv.cg > 1 ? nglob : 0) + t;
  }
  return true;
}

// Query blocks that attend key block k, by the whole calling wave: every block if k is global (Sec. 2:
// A(:, i) = 1 for i in G); else the global query blocks, the window, and the rows of rand_idx that name
// k (a ballot scan of the head's table).  Without the query blocks that were not computed (skip_q).
// Returns the count; one wave per workgroup writes the list.
__device__ __forceinline__ int build_query_list(const BwdParams& p, const Pattern& pat, int bi, int h, int k,
                                                int* jlist, bool write) {
  const int lane = lane_id();
  const bool key_global = pat.is_global(k);
  int cnt = 0;
  auto take = [&](bool valid, int j) {
    if (p.skip_q && valid) valid = block_has_valid_key(p.kmask, bi, p.n, j);
    const uint64_t m = __ballot(valid);
    const int rank = cnt + mask_rank(m);
    if (valid && write && rank < kMaxBwdBlocks) jlist[rank] = j;
    cnt += static_cast<int>(__popcll(m));
  };
  if (key_global) {
    for (int j0 = 0; j0 < p.nb; j0 += 64) take(j0 + lane < p.nb, j0 + lane);
  } else {
    for (int c0 = 0; c0 < p.g + p.w; c0 += 64) {
      const int ci = c0 + lane;
      const int j = ci < p.g ? pat.global_block(ci) : k - pat.half() + (ci - p.g);
      take(ci < p.g || (ci < p.g + p.w && j >= 0 && j < p.nb && !pat.is_global(j)), j);
    }
    if (p.rand_idx) {
      const int32_t* tbl = p.rand_idx + static_cast<size_t>(h) * p.nb * p.r;
      for (int j0 = 0; j0 < p.nb; j0 += 64) {
        const int j = j0 + lane;
        bool valid = false;
        if (j < p.nb && !pat.is_global(j) && !pat.in_window(j, k))
          for (int t = 0; t < p.r; ++t) valid |= tbl[static_cast<size_t>(j) * p.r + t] == k;
        take(valid, j);
      }
    }
  }
  return cnt < kMaxBwdBlocks ? cnt : kMaxBwdBlocks;  // (never more: the host bounds nb, a block is listed once)
}

// Enqueues: the dQ kernel (which also computes the row sums D), the dK/dV kernel and the
// fixed-order reductions.
int launch_bwd_bf16(const BwdParams& p, hipStream_t stream);

// The same for fp32 tensors (Q, K, V, O, dO fp32).
int launch_bwd_f32(const BwdParams& p, hipStream_t stream);

// Fixed-order sums of the partial gradients of both (nothing if no row and no column is split).
int launch_bwd_reduce(const BwdParams& p, hipStream_t stream);

}  // namespace bb
#endif  // BB_BWD_KERNELS_H_
