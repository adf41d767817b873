// Backward kernels (bf16 storage, fp32 gradients).  The paper gives no backward
// pass; this is the calculus of eq. (AT) of Sec. 2 on the blocked pattern of App. D.
// With P the row softmax recomputed from Q, K and the forward's LSE:
//   dV = P^T dO;  dP = dO V^T;  D_i = sum_c dO_ic O_ic;  dS = P o (dP - D);
//   dQ = scale dS K;  dK = scale dS^T Q.
//
// Two gather kernels, no atomics:
//   * bwd_dq_kernel walks the key-block list of a query block (the forward's
//     decomposition): S^T, dP^T and dS^T are [keys x queries] tiles, one lane per
//     query, and dQ^T += K^T dS^T.  It also computes the row sums D (and leaves them
//     in the workspace for the second kernel).
//   * bwd_dkv_kernel walks the query-block list of a key block -- the inverse of the
//     pattern (invert_pattern, part of the dQ launch) -- with S, dP, dS as
//     [queries x keys] tiles, one lane per key, dV^T += dO^T P and dK^T += Q^T dS.
// Lists longer than an item takes are cut into slices -- those of global blocks into 8 to 32 blocks each in large
// launches, longer or none in small ones (RowSplit, KeySplit) -- whose partial sums are added in slice order by
// bwd_reduce_kernel (bit-reproducible).
#include "bwd_kernels.h"
#include "key_list.h"
#include "tile_ops.h"

#include <cstdio>
#include <type_traits>

namespace bb {

namespace {

__device__ __forceinline__ void zero_acc(f32x16 (&a)[2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[t][r] = 0.f;
}

// Sum over each group of eight lanes, in all of them.
__device__ __forceinline__ float add_over_8_lanes(float x) {
  auto moved = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  x += moved(x, std::integral_constant<int, 0xB1>{});   // quad_perm [1, 0, 3, 2]
  x += moved(x, std::integral_constant<int, 0x4E>{});   // quad_perm [2, 3, 0, 1]
  x += moved(x, std::integral_constant<int, 0x141>{});  // row_half_mirror: the other four of the eight
  return x;
}

// The inverse of the pattern for one head and 64 key blocks: for a non-global key block the set of query
// blocks that attend it, as bits, and its place in the order of falling list length.  One wave; it runs
// beside the first dQ items, under whose time its own (5 us at nb = 64) disappears.  lds: 9 * kMaxBwdBlocks words.
__device__ __forceinline__ void invert_pattern(const BwdParams& p, const Pattern& pat, unsigned wg, uint32_t* lds) {
  const int groups = (p.nb + 63) / 64;
  const int h = wg / groups, group = wg % groups, lane = lane_id();
  if (h >= p.H) return;
  auto low_bits = [](int n) { return n <= 0 ? 0u : n >= 32 ? ~0u : (1u << n) - 1u; };
  uint32_t* const bits = lds;                                 // [key block][kSetWords]
  int* const len = reinterpret_cast<int*>(lds) + kMaxBwdBlocks * kSetWords;  // of its list; 0: global, or past the end
  const int first = pat.lead(), end = p.nb - pat.trail();     // non-global blocks
  for (int i = lane; i < kMaxBwdBlocks * kSetWords; i += 64) bits[i] = 0u;
  for (int i = lane; i < kMaxBwdBlocks; i += 64) len[i] = 0;
  asm volatile("" ::: "memory");
  // a lane per query block
  for (int j = lane; j < p.nb; j += 64) {
    const uint32_t bit = 1u << (j & 31);
    uint32_t* const col = bits + (j >> 5);
    if (!pat.is_global(j)) {
      const int lo = j - pat.half() > first ? j - pat.half() : first, hi = j + pat.half() < end - 1 ? j + pat.half() : end - 1;
      for (int k = lo; k <= hi; ++k) atomicOr(col + k * kSetWords, bit);
      if (p.rand_idx) {
        const int32_t* row = p.rand_idx + (static_cast<size_t>(h) * p.nb + j) * p.r;
#pragma unroll 4
        for (int t = 0; t < p.r; ++t) {
          const int k = row[t];
          if (k >= first && k < end) atomicOr(col + k * kSetWords, bit);
        }
      }
    }
  }
  asm volatile("" ::: "memory");
  for (int k = first + lane; k < end; k += 64) {
    int n = 0;
#pragma unroll
    for (int w = 0; w < kSetWords; ++w) {
      // the global query blocks: [0, first) and [end, nb)
      const uint32_t set = bits[k * kSetWords + w] | (low_bits(first - 32 * w) | (low_bits(p.nb - 32 * w) & ~low_bits(end - 32 * w)));
      bits[k * kSetWords + w] = set;
      n += __popc(set);
    }
    len[k] = n;
  }
  asm volatile("" ::: "memory");
  const int k = group * 64 + lane;
  const bool mine = k >= first && k < end;
  const int my_len = mine ? len[k] : 0;
  int rank = 0;
#pragma unroll 4
  for (int k4 = 0; k4 < p.nb; k4 += 4) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(len + k4);
#pragma unroll
    for (int u = 0; u < 4; ++u) rank += static_cast<int>(v[u]) + (k4 + u < k ? 1 : 0) > my_len ? 1 : 0;  // longer, or as long and before
  }
  if (mine) {
    p.key_order[h * p.nb + rank] = k;
    u32x4* dst = reinterpret_cast<u32x4*>(p.query_sets + (static_cast<size_t>(h) * p.nb + k) * kSetWords);
#pragma unroll
    for (int w = 0; w < kSetWords / 4; ++w) dst[w] = *reinterpret_cast<const u32x4*>(bits + k * kSetWords + w * 4);
  }
}

// Query blocks that attend key block k, by both waves of a workgroup (wave 0 writes the list), in
// ascending order: every block if k is global (Sec. 2: A(:, i) = 1 for i in G); else the set that
// invert_pattern left.  Without the query blocks that were not computed (skip_q).
__device__ __forceinline__ int query_list(const BwdParams& p, const Pattern& pat, int bi, int h, int k, int* jlist,
                                          bool write) {
  const int lane = lane_id();
  const bool key_global = pat.is_global(k);
  const uint32_t* set = p.query_sets + (static_cast<size_t>(h) * p.nb + k) * kSetWords;
  int cnt = 0;
  for (int j0 = 0; j0 < p.nb; j0 += 64) {
    const int j = j0 + lane;
    bool valid = j < p.nb;
    if (!key_global) valid = (set[j >> 5] >> (j & 31)) & 1;  // (bits past nb are 0)
    if (p.skip_q && valid) valid = block_has_valid_key(p.kmask, bi, p.n, j);
    const uint64_t m = __ballot(valid);
    if (valid && write) jlist[cnt + mask_rank(m)] = j;
    cnt += static_cast<int>(__popcll(m));
  }
  return cnt;
}

}  // namespace

// ---------------------------------------------------------------------------------------
// dQ: one work item = (batch*head, query block j, slice of j's key-block list), one wavefront per item
// ---------------------------------------------------------------------------------------
// A block pair is four units: 32 keys x 32 queries (query tile A or B), key half by key half.  Stages
// of unit u, in the order the wave issues them:
//   a(u)  S^T = K Q^T on the matrix pipe (4 MFMAs), beside dS(u-1) = P o (dP - D) and its conversion
//   b(u)  dP^T = V dO^T and dQ^T += K^T dS^T of unit u-1 (8 MFMAs), beside P = 2^(S^T c - LSE log2e)
// so that both pipes always have independent work, within the wave and between the two waves of a SIMD,
// which never wait for each other.
// Why this split: per block pair and compute unit the three products take the matrix pipes 384 cycles.
// Operands come from LDS, 128 bytes per cycle: a wave with 32 queries (two waves sharing the tiles, as
// this kernel was before) reads 48 KB per pair, 384 cycles more that nothing hid.  With 64 queries per
// wave every K, V and K^T fragment feeds two MFMAs: 24 KB.  Key halves, not whole blocks, because 64
// keys' worth of fragments do not fit beside Q, dO and dQ (128 registers).
// What bounds it now: issue slots of the vector port (an MFMA takes 17 cycles of it, an exponential 7 to 9,
// a conversion 5, other instructions 3, measured with two waves per SIMD: 2080 per block pair and SIMD
// against 1536 of the matrix pipe; 2300 are reached) and, with all waves of a launch of 1872 items resident
// at once, the start: Q, dO, O tiles of every item together, 9 k of a wave's 41 k cycles.
// In back-to-back steps, 24 slices, n = 4096: 37 -> 34 us; 16 of n = 16384: 92 -> 83; n = 3072, 48 slices,
// dropout: 49 -> 47.
struct DqState {
  bf16x8 qb[2][4], dob[2][4];  // B operands of the item: Q^T, dO^T (lane = query, d = 16ks + 8hf .. +8)
  f32x16 dq[2][2];             // [query tile][d tile]
  bf16x8 ka[4], va[4];         // straight fragments of the key half in work
  bf16x8 kt[2][2];             // its transposed K fragments (until the next half's arrive)
  f32x16 s, dp;                // the unit in work
  float lse2[2], d[2];         // per query tile: LSE log2(e) of this lane's query, its row sum D
};

// kDrop: attention dropout, dP = M / (1 - p) o (dO V^T) with M the keep mask (a second instance of
// the kernel, so that the one without dropout keeps its registers and its schedule).

// dS of the previous unit (query tile q), packed as B operand.
template <bool kDrop>
__device__ __forceinline__ void dq_ds(const DqState& st, const f32x16& p, const f32x16& dp, int q,
                                      const Dropout& drop, uint32_t drop_rk, const uint32_t* drop_words,
                                      bf16x8 (&dsb)[2]) {
  const float d = st.d[q];
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    float x0, x1;
    if constexpr (kDrop) {
      // registers r, r + 1 are keys 2m, 2m + 1: one word of the mask
      const uint32_t wd = drop_doubled(drop_rk ^ drop_words[r >> 1]);
      x0 = drop_keep_low(wd, drop.thr) ? __builtin_fmaf(dp[r], drop.rs, -d) : -d;
      x1 = drop_keep_high(wd, drop.thr) ? __builtin_fmaf(dp[r + 1], drop.rs, -d) : -d;
    } else {
      x0 = dp[r] - d;
      x1 = dp[r + 1] - d;
    }
    const bf16x2 pk = {static_cast<__bf16>(p[r] * x0), static_cast<__bf16>(p[r + 1] * x1)};
    dsb[r >> 3][r & 7] = pk[0];
    dsb[r >> 3][(r & 7) + 1] = pk[1];
  }
}

// Issue order of stage a: per MFMA a quarter of the vector work and of the LDS reads; of stage b: per
// MFMA two exponentials.
template <int DS_READS, int VALU>
__device__ __forceinline__ void pin_a() {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, DS_READS / 4, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}
template <int DS_READS>
__device__ __forceinline__ void pin_b() {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (u < DS_READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// kWaves: waves of a workgroup.  Large launches: 1, every wave an item of its own.  Smaller ones: 2 (dq_two_waves)
// or 4 (p.by_row), which deal out the list of one item among themselves and add their shares of dQ in LDS.
template <bool kDrop, int kWaves>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2)))
void bwd_dq_kernel(BwdParams p) {
  // K and V tiles of the block in work, then swapped: what takes a half's place is requested as soon as
  // the half sits in registers, the next block's K half where the V half was (free first) and its V half
  // where the K half was, so that every request has one and a half halves of a block to land
  __shared__ __attribute__((aligned(1024))) char lds_all[kWaves][2][kTile];
  __shared__ int klist_all[kWaves][kChunkMax];
  __shared__ uint32_t key_bits_all[kWaves][kChunkMax][2];  // validity of the keys of blocks with padded keys inside
  __shared__ float dvals_all[kWaves][kBlk];
  __shared__ __attribute__((aligned(16))) uint32_t drop_words_all[kDrop ? kWaves : 1][2][32];  // key words of two blocks in turn
  const int wv = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char (&lds)[2][kTile] = lds_all[wv];
  int* const klist = klist_all[wv];
  uint32_t (*const key_bits)[2] = key_bits_all[wv];
  float* const dvals = dvals_all[wv];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  WorkItem it;
  // the first workgroups make the inverse of the pattern for the dK/dV kernel, which runs after this one
  if (blockIdx.x < p.inverse_wgs) {
    if (wv == 0) invert_pattern(p, pat, blockIdx.x, reinterpret_cast<uint32_t*>(lds));
    return;
  }
  if (!decode_item(p.split, pat, p.BH, blockIdx.x - p.inverse_wgs, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id();
  const int hf = lane >> 5, col = lane & 31;
  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;

  // Q and dO tiles into LDS, the O tile into registers (8 lanes a row), all in one trip to memory, whole
  // rows at a time: fetched in operand layout these loads touch every row in each instruction, and all
  // waves of the launch start with them.
  const unsigned lds_a = __builtin_amdgcn_readfirstlane(lds_addr(lds[0]));
  unsigned voff[2];
  half_load_offsets(lane, voff);
  const size_t row0 = bh_row0 + static_cast<size_t>(it.j) * kBlk;
  tile_load_async_wave(static_cast<const char*>(p.Q) + row0 * (kDim * 2), lds_a, voff);
  tile_load_async_wave(static_cast<const char*>(p.dO) + row0 * (kDim * 2), lds_a + kTile, voff);
  bf16x8 orow[8];  // rows 8 ii + lane / 8, columns 8 (lane % 8) .. + 7
#pragma unroll
  for (int ii = 0; ii < 8; ++ii)
    orow[ii] = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(p.O) + row0 * kDim)[ii * 64 + lane];
  float lse = p.LSE[row0 + lane];

  // a query block that the forward did not compute (no valid position, and the caller asked for
  // such blocks to be skipped): no key block, D = 0, probabilities 0
  const bool skip = p.skip_q && !block_any_valid_scalar(p.kmask, bi, p.n, it.j);
  KeyList list = item_key_list<true>(pat, p.rand_idx, p.r, p.kmask, p.n, bi, h, it.j, it.row_global,
                                     it.chunk * it.len + wv * (it.len / kWaves), it.len / kWaves, lane, klist, key_bits);
  const int cnt = __builtin_amdgcn_readfirstlane(skip ? 0 : list.cnt);
  const int kl = list.entry;
  const unsigned partial = __builtin_amdgcn_readfirstlane(list.partial);

  const char* kbase = static_cast<const char*>(p.K) + bh_row0 * (kDim * 2);
  const char* vbase = static_cast<const char*>(p.V) + bh_row0 * (kDim * 2);
  // (past the end of the list: its last block again, which nobody uses)
  auto tile_off = [&](int i) {
    return static_cast<size_t>(__builtin_amdgcn_readlane(kl, i < cnt ? i : cnt - 1)) * kTile;
  };

  const StraightOffsets so(lane);
  DqState st;
  wait_tile_loads<0>();
  so.read(lds[0], st.qb);
  so.read(lds[1], st.dob);
  // D_i = sum_c dO_ic O_ic: row by row, an eighth of a row per lane, added up over the eight lanes
  float dsum = 0.f;
#pragma unroll
  for (int ii = 0; ii < 8; ++ii) {
    const bf16x8 g = *reinterpret_cast<const bf16x8*>(lds[1] + tile_off_bf16(ii * 8 + (lane >> 3), lane & 7));
    float part = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) part = __builtin_fmaf(static_cast<float>(g[e]), static_cast<float>(orow[ii][e]), part);
    part = add_over_8_lanes(part);
    if ((lane & 7) == ii) dsum = part;
  }
  wait_lds_reads();
  if (cnt > 0) {
    const size_t off = tile_off(0);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      half_load_async(kbase + off, lds_a, hh, voff);
      half_load_async(vbase + off, lds_a + kTile, hh, voff);
    }
  }
  // (+inf where the forward found no valid key, so that the recomputed probabilities of such a row are
  // 0.)  The first slice of a row also leaves D and LSE log2(e) in the workspace for the dK/dV kernel,
  // which runs after this one.
  if (skip) dsum = 0.f;
  lse = (skip || lse == neg_inf()) ? __builtin_inff() : lse * kLog2e;
  dvals[(lane & 7) * 8 + (lane >> 3)] = dsum;
  asm volatile("" ::: "memory");
  if (it.chunk == 0 && wv == 0) {
    p.Dvec[row0 + lane] = -dvals[lane];  // negated: the other kernel starts its dP accumulators from it
    p.Lvec[row0 + lane] = lse;
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    st.d[q] = dvals[q * 32 + col];
    st.lse2[q] = __shfl(lse, q * 32 + col);
    zero_acc(st.dq[q]);
  }
  asm volatile("" : "+v"(st.d[0]), "+v"(st.d[1]), "+v"(st.lse2[0]), "+v"(st.lse2[1]));
  uint32_t drop_rk[2] = {0u, 0u};
  if constexpr (kDrop) {
#pragma unroll
    for (int q = 0; q < 2; ++q) drop_rk[q] = drop_first(drop_row_key(p.drop, static_cast<uint32_t>(row0 + q * 32 + col)));
  }

  const TransposedOffsets to(lane);
  const float c = p.c;

  if (cnt > 0) {
    // what the first unit "finishes": nothing
#pragma unroll
    for (int r = 0; r < 16; ++r) st.s[r] = st.dp[r] = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) st.kt[a][b][e] = static_cast<__bf16>(0.f);
    wait_tile_loads<8>();  // K(0).h0, V(0).h0 (each request is four loads)
    read_straight_half(so, lds[0], 0, st.ka);

    // dS of the last unit, its share of dQ in stage b of the next
    bf16x8 dsb[2];
    auto mask_ds = [&](int i, int hh) {
      if ((partial >> i) & 1) drop_padded_keys(key_bits[i][hh], hf, dsb);
    };
    auto dq_update = [&](int q) {
#pragma unroll
      for (int sgl = 0; sgl < 2; ++sgl)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          st.dq[q][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.kt[dt][sgl], dsb[sgl], st.dq[q][dt], 0, 0, 0);
    };
    auto products = [&](const bf16x8 (&a)[4], const bf16x8 (&b)[4], f32x16& acc) {
      f32x16 z;
#pragma unroll
      for (int r = 0; r < 16; ++r) z[r] = 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], z, 0, 0, 0);
#pragma unroll
      for (int ks = 1; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], b[ks], acc, 0, 0, 0);
    };
    // dP of query tile q beside the dQ products of the other one, alternating: an MFMA that adds to the
    // result of the one before it waits for it
    auto products_and_update = [&](int q, int qu) {
      f32x16 z;
#pragma unroll
      for (int r = 0; r < 16; ++r) z[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        st.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.va[ks], st.dob[q][ks], ks == 0 ? z : st.dp, 0, 0, 0);
        st.dq[qu][ks & 1] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.kt[ks & 1][ks >> 1], dsb[ks >> 1], st.dq[qu][ks & 1], 0, 0, 0);
      }
    };
    auto probabilities = [&](int q) {
#pragma unroll
      for (int r = 0; r < 16; ++r) st.s[r] = fast_exp2(__builtin_fmaf(st.s[r], c, -st.lse2[q]));
    };

    // block i; its K tile is lds[X], its V tile lds[X ^ 1]
    auto block = [&](int i, auto X) {
      constexpr int kx = decltype(X)::value;
      if constexpr (kDrop)
        drop_key_words(drop_words_all[wv][kx], static_cast<uint32_t>(__builtin_amdgcn_readlane(kl, i)), lane_again(lane));
      const size_t off1 = tile_off(i + 1);
      const char* k1 = kbase + off1;
      const char* v1 = vbase + off1;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        // key words of the previous unit's half (tile B of the half before this one) and of this one
        const uint32_t* const words_prev = drop_unit_words(drop_words_all[kDrop ? wv : 0][hh ? kx : kx ^ 1], hh ^ 1, hf);
        const uint32_t* const words_cur = drop_unit_words(drop_words_all[kDrop ? wv : 0][kx], hh, hf);
        f32x16 s_new;
        // ---- a(A): V fragments of this half (the two requests after it are still out)
        wait_tile_loads<8>();
        read_straight_half(so, lds[kx ^ 1], hh, st.va);
        products(st.ka, st.qb[0], s_new);
        dq_ds<kDrop>(st, st.s, st.dp, 1, p.drop, drop_rk[1], words_prev, dsb);
        pin_a<4, 10>();
        mask_ds(hh ? i : (i > 0 ? i - 1 : 0), hh ^ 1);
        st.s = s_new;
        // ---- b(A): the V half is in registers, its place takes the next block's K half
        wait_lds_reads();
        half_load_async(k1, lds_a + (kx ^ 1) * kTile, hh, voff);
        products_and_update(0, 1);
        probabilities(0);
        pin_b<0>();
        // ---- a(B)
        read_transposed_half(to, lds[kx], hh, st.kt);
        products(st.ka, st.qb[1], s_new);
        dq_ds<kDrop>(st, st.s, st.dp, 0, p.drop, drop_rk[0], words_cur, dsb);
        pin_a<8, 10>();
        mask_ds(i, hh);
        st.s = s_new;
        // ---- b(B): the K half likewise; the next half's K has landed (two younger requests)
        wait_lds_reads();
        wait_tile_loads<8>();
        half_load_async(v1, lds_a + kx * kTile, hh, voff);
        read_straight_half(so, lds[hh ? kx ^ 1 : kx], hh ^ 1, st.ka);
        products_and_update(1, 0);
        probabilities(1);
        pin_b<4>();
      }
    };
    for (int i = 0; i < cnt; i += 2) {
      block(i, std::integral_constant<int, 0>{});
      if (i + 1 < cnt) block(i + 1, std::integral_constant<int, 1>{});
    }
    // the last unit's dS and its share of dQ
    dq_ds<kDrop>(st, st.s, st.dp, 1, p.drop, drop_rk[1], drop_unit_words(drop_words_all[kDrop ? wv : 0][(cnt - 1) & 1], 1, hf), dsb);
    mask_ds(cnt - 1, 1);
    dq_update(1);
    wait_tile_loads<0>();  // requests past the end of the list
  }

  // dQ^T accumulators, turned through LDS so that memory sees whole rows
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = st.dq[q][dt][r4 * 4 + e] * p.scale;
        *reinterpret_cast<f32x4*>(lds[dt] + tile_off_bf16(q * 32 + col, r4 * 2 + hf)) = v;
      }
  wait_lds_reads();
  if constexpr (kWaves > 1) __syncthreads();
  float* dst = it.nchunks == 1 ? p.dQ + row0 * kDim : p.part_dq + static_cast<size_t>(it.slot) * (kBlk * kDim);
#pragma unroll
  for (int ii = 0; ii < 16 / kWaves; ++ii) {
    const int row = (wv * (16 / kWaves) + ii) * 4 + (lane >> 4), cc = lane & 15;
    f32x4 v = *reinterpret_cast<const f32x4*>(lds_all[0][cc >> 3] + tile_off_bf16(row, cc & 7));
#pragma unroll
    for (int u = 1; u < kWaves; ++u) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(lds_all[u][cc >> 3] + tile_off_bf16(row, cc & 7));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += x[e];
    }
    *reinterpret_cast<f32x4*>(dst + row * kDim + cc * 4) = v;
  }
}

// ---------------------------------------------------------------------------------------
// dK, dV: one work item = (batch*head, key block k[, slice of its query-block list]), two waves
// ---------------------------------------------------------------------------------------
// Wave wv owns 32 keys of the block; the list's Q and dO tiles come in halves of 32 queries through a ring
// of four places in LDS that both waves read, one barrier per half.  Stages of half h, in issue order:
//   A(h)  dK^T += Q^T dS of half h-1 and dP = dO V^T (8 MFMAs), beside P = 2^(S c - LSE log2e) and its conversion
//   B(h)  dV^T += dO^T P and S = Q K^T of half h+1 (8 MFMAs), beside dS = P o dP and its conversion
// dP starts from -D, staged with the tiles (element r of an accumulator belongs to query row acc_row(r)), and
// LSE log2(e) rides in the fma that scales S, so neither subtraction costs a vector instruction.  (S does not
// start from -LSE / scale: that rounds every product at the size of LSE / scale, and overflows for small scales.)  Operands are read from LDS one
// stage before their use; a half is requested three halves ahead.
// What bounds it: issue slots of the vector port, where an MFMA takes 17 cycles, an exponential 7 to 9, a
// conversion 5 and other instructions 3 (measured, two waves per SIMD): 2340 cycles per block pair and
// SIMD against 2048 of the matrix pipe.  One wave alone reaches
// 1950, two on a SIMD 2700 (per pair; 3220 when a pair was one stage after the other).
// Items run longest list first (key_order of the workspace): the lists of the non-global key blocks hold 5
// to 16 query blocks at the base pattern, and in the order of the sequence the launch ended on whichever
// came last.  In back-to-back steps, 24 slices, n = 4096: 46 -> 40 us; 16 of n = 16384: 120 -> 103; 48 of n = 3072
// with padding and dropout, where two neighbouring keys share the words of the keep mask (one per 2 x 1
// elements): 61 -> 50.
//
// kDrop: attention dropout (see bwd_dq_kernel): dV takes the kept probabilities (rescaled at the
// end), dP is masked and rescaled before D is subtracted.  The row keys of the mask for the queries of a
// half are staged in LDS beside LSE and D.
constexpr int kRing = 4;
constexpr int kDkvThreads = 128;

template <int DS_READS, int VALU>
__device__ __forceinline__ void pin_half_stage() {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, DS_READS / 8, 0);
    if (VALU == 0)
      __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);  // two exponentials
    else
      __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// kTeams: pairs of waves of a workgroup, each with a ring of its own.  Large launches: 1.  Smaller ones: 2 (dkv_two_teams)
// or 4 (p.by_row), which deal out the item's list and add their shares of dK and dV in LDS.
template <bool kDrop, int kTeams>
__global__ __launch_bounds__(kDkvThreads * kTeams) __attribute__((amdgpu_waves_per_eu(2)))
void bwd_dkv_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char ring_all[kTeams][kRing][2][kHalfTile];  // Q half, dO half
  __shared__ __attribute__((aligned(256))) float lds_l_all[kTeams][kRing][kBlk];         // LSE log2(e) of the whole block
  __shared__ __attribute__((aligned(256))) float lds_d_all[kTeams][kRing][kBlk];         // -D
  __shared__ __attribute__((aligned(256))) uint32_t lds_rk_all[kTeams][kDrop ? kRing : 1][kBlk];
  __shared__ int jlist[kMaxBwdBlocks];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  KeyItem it;
  if (!decode_key_item(p, pat, blockIdx.x, &it)) return;
  const int bh = it.bh;
  const int bi = bh / p.H, h = bh % p.H;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = wave & 1, team = kTeams == 1 ? 0 : wave >> 1;
  auto& ring = ring_all[team];
  auto& lds_l = lds_l_all[team];
  auto& lds_d = lds_d_all[team];
  auto& lds_rk = lds_rk_all[team];
  const int hf = lane >> 5, col = lane & 31;
  if (!it.key_global) it.k = p.key_order[h * p.nb + it.k - pat.lead()];
  const int k = __builtin_amdgcn_readfirstlane(it.k);

  const size_t bh_row0 = static_cast<size_t>(bh) * p.n;
  const size_t krow0 = bh_row0 + static_cast<size_t>(k) * kBlk + wv * 32;  // first of this wave's keys
  float* dk_dst = it.nchunks == 1 ? p.dK + krow0 * kDim
                                  : p.part_dk + static_cast<size_t>(it.slot) * (kBlk * kDim) + wv * 32 * kDim;
  float* dv_dst = it.nchunks == 1 ? p.dV + krow0 * kDim
                                  : p.part_dv + static_cast<size_t>(it.slot) * (kBlk * kDim) + wv * 32 * kDim;

  unsigned voff[2];
  half_load_offsets(lane, voff);
  const unsigned ring_a = __builtin_amdgcn_readfirstlane(lds_addr(ring));
  // this wave's keys' K and V rows, through places 2 and 3 of the ring (whole rows at a time)
  {
    const size_t off = krow0 * (kDim * 2);
    half_load_async(static_cast<const char*>(p.K) + off, ring_a + (2 * 2 + wv) * kHalfTile, 0, voff);
    half_load_async(static_cast<const char*>(p.V) + off, ring_a + (3 * 2 + wv) * kHalfTile, 0, voff);
  }
  uint64_t vbits = ~0ull;
  if (p.kmask) vbits = key_valid_bits(p.kmask, bi, p.n, k);
  const int total = vbits == 0 ? 0 : query_list(p, pat, bi, h, k, jlist, wave == 0);
  // this team's share: entries chunk, chunk + nchunks, ... of the list
  const int chunk = it.chunk * kTeams + team, nchunks = it.nchunks * kTeams;
  auto share = [&](int c) { return __builtin_amdgcn_readfirstlane(c < total ? (total - c + nchunks - 1) / nchunks : 0); };
  const int cnt = share(chunk);
  __syncthreads();

  f32x16 dk[2], dv[2];
  zero_acc(dk);
  zero_acc(dv);
  if (cnt > 0) {
    const char* qbase = static_cast<const char*>(p.Q) + bh_row0 * (kDim * 2);
    const char* dobase = static_cast<const char*>(p.dO) + bh_row0 * (kDim * 2);
    const char* tbase = wv == 0 ? qbase : dobase;  // wave 0 brings the Q halves and LSE, wave 1 dO and D
    const float* vecbase = (wv == 0 ? p.Lvec : p.Dvec) + bh_row0;
    const unsigned vec_a = __builtin_amdgcn_readfirstlane(wv == 0 ? lds_addr(lds_l) : lds_addr(lds_d));
    // (past the end of the list: its last entry again, which nobody uses)
    auto entry = [&](int hh) {
      const int i = hh >> 1;
      return jlist[chunk + (i < cnt ? i : cnt - 1) * nchunks];
    };
    // five loads per wave and half
    auto request = [&](int hh, int j_, int place) {
      const int j = __builtin_amdgcn_readfirstlane(j_);
      half_load_async(tbase + static_cast<size_t>(j) * kTile + (hh & 1) * kHalfTile, ring_a + (place * 2 + wv) * kHalfTile, 0,
                      voff);
      vec_load_async(vecbase + static_cast<size_t>(j) * kBlk, vec_a + place * (kBlk * 4), lane);
      if constexpr (kDrop) {
        if (wv == 0)
          lds_rk[place][lane] = drop_first(drop_row_key(p.drop, static_cast<uint32_t>(bh_row0 + static_cast<size_t>(j) * kBlk + lane)));
      }
    };
    request(0, entry(0), 0);
    request(1, entry(1), 1);

    // B operands kept for the whole item: K^T and V^T, lane = key `col`, d = 16ks + 8hf .. +8
    const StraightOffsets so(lane);
    const TransposedOffsets to(lane);
    bf16x8 kb[4], vb[4];
    wait_tile_loads<10>();
    read_straight_half(so, ring[2][wv], 0, kb);
    read_straight_half(so, ring[3][wv], 0, vb);
    wait_lds_reads();
    wait_tile_loads<5>();
    BB_BARRIER();
    request(2, entry(2), 2);

    const float c = p.c;
    bf16x8 qs[4], dos[4], qt[2][2], dot[2][2], pb[2], dsb[2];
    f32x16 s, dp, lse;  // (lse: the elements of the staged vector that belong to s)
    // the rows of an accumulator, from a staged vector
    auto start_from = [&](const float* vec, f32x16& acc) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(vec + acc_row(r4 * 4, hf));
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[r4 * 4 + e] = v[e];
      }
    };
    auto add_products = [&](const bf16x8 (&a)[4], const bf16x8 (&b)[4], f32x16& acc) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], b[ks], acc, 0, 0, 0);
    };
    auto add_transposed = [&](const bf16x8 (&a)[2][2], const bf16x8 (&b)[2], f32x16 (&acc)[2]) {
#pragma unroll
      for (int sgl = 0; sgl < 2; ++sgl)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[dt][sgl], b[sgl], acc[dt], 0, 0, 0);
    };
    auto pack = [&](const f32x16& x, bf16x8 (&b)[2]) {
#pragma unroll
      for (int r = 0; r < 16; ++r) b[r >> 3][r & 7] = static_cast<__bf16>(x[r]);
    };
    // S of half 0; what A(0) "finishes": nothing
    read_straight_half(so, ring[0][0], 0, qs);
    start_from(lds_l[0], lse);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
    add_products(qs, kb, s);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
      for (int e = 0; e < 8; ++e) dsb[a][e] = static_cast<__bf16>(0.f);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) qt[a][b][e] = static_cast<__bf16>(0.f);
    }
    // (dropout) this lane's key: its pair's share of the words' argument, its half of a word
    const uint32_t my_pair = drop_first((static_cast<uint32_t>(k * kBlk + wv * 32 + col) >> 1) * kDropPairStep);
    const int odd = col & 1, my_shift = odd * 16;
    const uint32_t drop_thr = kDrop ? drop_pair_threshold(p.drop) : 0u;
    // keep bits of this lane's key, bit r: the query of accumulator register r.  A word of the mask serves two
    // keys, neighbouring lanes: the even one makes those of registers 0 .. 7, the odd one those of 8 .. 15
    auto keep_bits = [&](const uint32_t* row_keys) {
      uint32_t both = 0;  // bit i: even key, 16 + i: odd key
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const u32x4 k4 = *reinterpret_cast<const u32x4*>(row_keys + odd * 16 + acc_row(u * 4, hf));
#pragma unroll
        for (int e = 0; e < 4; ++e)
          both |= drop_keep_pair(drop_doubled(k4[e] ^ my_pair), drop_thr) << (u * 4 + e);
      }
      const uint32_t other = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(both), 0xB1, 0xf, 0xf, true));  // quad_perm [1, 0, 3, 2]
      const uint32_t mine = (both >> my_shift) & 0xffu, theirs = (other >> my_shift) & 0xffu;
      return odd ? theirs | mine << 8 : mine | theirs << 8;
    };

    int j_next = entry(3);
    auto half = [&](int hh, auto P) {
      constexpr int here = decltype(P)::value, next = (here + 1) % kRing, row = (here & 1) * 32, row1 = row ^ 32;
      // everything this wave read of half h-1 is in registers and its share of half h+1 has landed; after
      // the barrier that holds for both waves, and half h+3 takes the place of half h-1
      wait_lds_reads();
      wait_tile_loads<5>();
      BB_BARRIER();
      request(hh + 3, j_next, (here + 3) % kRing);

      // ---- A(h)
      read_straight_half(so, ring[here][1], 0, dos);
      if constexpr (kDrop) {
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] = 0.f;
      } else {
        start_from(lds_d[here] + row, dp);
      }
      read_transposed_half(to, ring[here][1], 0, dot);
      add_transposed(qt, dsb, dk);
      add_products(dos, vb, dp);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = fast_exp2(__builtin_fmaf(s[r], c, -lse[r]));
      if constexpr (kDrop) {
        // this lane's key against the queries of its accumulator rows: the kept probabilities go to dV,
        // and dP becomes M / (1 - p) o dP - D  (the staged vector holds -D)
        __builtin_amdgcn_sched_barrier(0);
        const float rs = p.drop.rs;
        const int keep = static_cast<int>(keep_bits(lds_rk[here] + row));
        f32x16 sk;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(lds_d[here] + row + acc_row(r4 * 4, hf));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int m = __builtin_amdgcn_sbfe(keep, r4 * 4 + e, 1);  // 0 or ~0
            sk[r4 * 4 + e] = __int_as_float(__float_as_int(s[r4 * 4 + e]) & m);
            dp[r4 * 4 + e] = __builtin_fmaf(__int_as_float(__float_as_int(dp[r4 * 4 + e]) & m), rs, d4[e]);
          }
        }
        pack(sk, pb);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        pack(s, pb);
        pin_half_stage<16, 0>();
      }

      // ---- B(h)
      f32x16 s_new;
      read_straight_half(so, ring[next][0], 0, qs);
      start_from(lds_l[next] + row1, lse);
#pragma unroll
      for (int r = 0; r < 16; ++r) s_new[r] = 0.f;
      read_transposed_half(to, ring[here][0], 0, qt);
      j_next = entry(hh + 4);
      add_transposed(dot, pb, dv);
      add_products(qs, kb, s_new);
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[r] *= s[r];
      pack(dp, dsb);
      pin_half_stage<16, 3>();
      s = s_new;
    };
    for (int hh = 0; hh < 2 * cnt; hh += 4) {
      half(hh, std::integral_constant<int, 0>{});
      half(hh + 1, std::integral_constant<int, 1>{});
      if (hh + 2 < 2 * cnt) {
        half(hh + 2, std::integral_constant<int, 2>{});
        half(hh + 3, std::integral_constant<int, 3>{});
      }
    }
    add_transposed(qt, dsb, dk);  // the last half's share
  }
  if constexpr (kTeams > 1) {  // the barriers of the team with the most entries, the first
    const int most = share(it.chunk * kTeams);
    for (int u = cnt > 0 ? 2 * cnt : (most > 0 ? -1 : 0); u < 2 * most; ++u) BB_BARRIER();
  }
  wait_tile_loads<0>();  // requests past the end of the list (with an empty one: K and V)
  __syncthreads();       // nobody reads the ring any more

  // gradients of a padded key are exactly 0 (selected, not multiplied: what was summed for it may be anything); turned
  // through LDS so that memory sees whole rows: this wave's 32 rows of dK, then of dV, d 0 .. 31 and 32 .. 63
  const bool key_valid = (vbits >> (wv * 32 + col)) & 1;
  const float vscale = kDrop ? p.drop.rs : 1.f;
  char* const out = &ring[0][0][0] + wv * (4 * kHalfTile);  // a team's ring is twice that
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      f32x4 a, b;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = key_valid ? dk[dt][r4 * 4 + e] * p.scale : 0.f;
        b[e] = key_valid ? dv[dt][r4 * 4 + e] * vscale : 0.f;
      }
      const int off = tile_off_bf16(col, r4 * 2 + hf);
      *reinterpret_cast<f32x4*>(out + dt * kHalfTile + off) = a;
      *reinterpret_cast<f32x4*>(out + (2 + dt) * kHalfTile + off) = b;
    }
  wait_lds_reads();
  if constexpr (kTeams > 1) __syncthreads();
#pragma unroll
  for (int ii = 0; ii < 8 / kTeams; ++ii) {
    const int row = (team * (8 / kTeams) + ii) * 4 + (lane >> 4), cc = lane & 15;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
    for (int u = 0; u < kTeams; ++u) {
      const char* src = &ring_all[u][0][0][0] + wv * (4 * kHalfTile) + (cc >> 3) * kHalfTile + tile_off_bf16(row, cc & 7);
      const f32x4 x = *reinterpret_cast<const f32x4*>(src), y = *reinterpret_cast<const f32x4*>(src + 2 * kHalfTile);
      if (u == 0) {
        a = x;
        b = y;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] += x[e];
          b[e] += y[e];
        }
      }
    }
    *reinterpret_cast<f32x4*>(dk_dst + row * kDim + cc * 4) = a;
    *reinterpret_cast<f32x4*>(dv_dst + row * kDim + cc * 4) = b;
  }
}

// ---------------------------------------------------------------------------------------
// Fixed-order sums of the partial gradients of split rows (dQ) and split columns (dK, dV)
// ---------------------------------------------------------------------------------------
// One launch covers all three: blocks [0, nq) are the dQ blocks of split query rows, then
// come the dK and the dV blocks of split key blocks.  Four workgroups per 64x64 block,
// thread t owns 4 columns of row part*16 + t/16.
__global__ __launch_bounds__(256) void bwd_reduce_kernel(BwdParams p, int nq_blocks, int nkv_blocks) {
  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  const int part = blockIdx.x & 3;
  int blk = blockIdx.x >> 2;
  const float* src;
  float* dst;
  int nslices;
  if (blk < nq_blocks) {
    const RowSplit& s = p.split;
    const int nglob_rows = s.cg > 1 ? p.g : 0;
    const int nsparse_rows = s.cs > 1 ? p.nb - p.g : 0;
    const int rows_per_bh = nglob_rows + nsparse_rows;
    const int bh = blk / rows_per_bh, rr = blk % rows_per_bh;
    int j, slot0;
    if (rr < nglob_rows) {
      j = pat.global_block(rr);
      nslices = s.cg;
      slot0 = bh * s.slots_per_bh + rr * s.cg;
    } else {
      const int t = rr - nglob_rows;
      j = pat.sparse_block(t);
      nslices = s.cs;
      slot0 = bh * s.slots_per_bh + (s.cg > 1 ? p.g * s.cg : 0) + t * s.cs;
    }
    src = p.part_dq + static_cast<size_t>(slot0) * (kBlk * kDim);
    dst = p.dQ + (static_cast<size_t>(bh) * p.n + j * kBlk) * kDim;
  } else {
    blk -= nq_blocks;
    const bool is_dv = blk >= nkv_blocks;
    if (is_dv) blk -= nkv_blocks;
    const KeySplit& s = p.kv;
    const int nglob_cols = s.cg > 1 ? p.g : 0;
    const int cols_per_bh = nglob_cols + (s.cs > 1 ? p.nb - p.g : 0);
    const int bh = blk / cols_per_bh, cc = blk % cols_per_bh;
    int k, slot0;
    if (cc < nglob_cols) {
      k = pat.global_block(cc);
      nslices = s.cg;
      slot0 = bh * s.slots_per_bh + cc * s.cg;
    } else {
      const int t = cc - nglob_cols;
      k = pat.sparse_block(t);
      nslices = s.cs;
      slot0 = bh * s.slots_per_bh + (s.cg > 1 ? p.g * s.cg : 0) + t * s.cs;
    }
    src = (is_dv ? p.part_dv : p.part_dk) + static_cast<size_t>(slot0) * (kBlk * kDim);
    dst = (is_dv ? p.dV : p.dK) + (static_cast<size_t>(bh) * p.n + k * kBlk) * kDim;
  }
  const int off = (part * 16 + (threadIdx.x >> 4)) * kDim + (threadIdx.x & 15) * 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 8;
  for (int c0 = 0; c0 < nslices; c0 += U) {
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cidx = c0 + u < nslices ? c0 + u : nslices - 1;
      v[u] = *reinterpret_cast<const f32x4*>(src + static_cast<size_t>(cidx) * (kBlk * kDim) + off);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c0 + u < nslices) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += v[u][e];
      }
  }
  *reinterpret_cast<f32x4*>(dst + off) = acc;
}

namespace {
bool launch_failed(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return false;
  fprintf(stderr, "bigbird: launch of %s failed: %s\n", what, hipGetErrorString(e));
  return true;
}
}  // namespace

int launch_bwd_bf16(const BwdParams& p, hipStream_t stream) {
  const unsigned qgrid = p.inverse_wgs + DieItems(p.BH, p.split.items_per_bh).grid();
  const bool drop = p.drop.thr != 0;
  const auto dq = p.dq_waves == kRowWaves ? (drop ? bwd_dq_kernel<true, kRowWaves> : bwd_dq_kernel<false, kRowWaves>)
                  : p.dq_waves == 2       ? (drop ? bwd_dq_kernel<true, 2> : bwd_dq_kernel<false, 2>)
                                          : (drop ? bwd_dq_kernel<true, 1> : bwd_dq_kernel<false, 1>);
  hipLaunchKernelGGL(dq, dim3(qgrid), dim3(64 * p.dq_waves), 0, stream, p);
  if (launch_failed("bwd_dq_kernel")) return BB_ERR_LAUNCH;
  const unsigned kvgrid = DieItems(p.BH, p.kv.items_per_bh).grid();
  const auto dkv = p.dkv_teams == kRowWaves ? (drop ? bwd_dkv_kernel<true, kRowWaves> : bwd_dkv_kernel<false, kRowWaves>)
                   : p.dkv_teams == 2       ? (drop ? bwd_dkv_kernel<true, 2> : bwd_dkv_kernel<false, 2>)
                                            : (drop ? bwd_dkv_kernel<true, 1> : bwd_dkv_kernel<false, 1>);
  hipLaunchKernelGGL(dkv, dim3(kvgrid), dim3(kDkvThreads * p.dkv_teams), 0, stream, p);
  if (launch_failed("bwd_dkv_kernel")) return BB_ERR_LAUNCH;

  return launch_bwd_reduce(p, stream);
}

int launch_bwd_reduce(const BwdParams& p, hipStream_t stream) {
  const RowSplit& s = p.split;
  const int rows_per_bh = (s.cg > 1 ? p.g : 0) + (s.cs > 1 ? p.nb - p.g : 0);
  const int cols_per_bh = (p.kv.cg > 1 ? p.g : 0) + (p.kv.cs > 1 ? p.nb - p.g : 0);
  const int nq_blocks = p.BH * rows_per_bh, nkv_blocks = p.BH * cols_per_bh;
  const int total = nq_blocks + 2 * nkv_blocks;
  if (total > 0) {
    hipLaunchKernelGGL(bwd_reduce_kernel, dim3(static_cast<unsigned>(total) * 4), dim3(256), 0, stream, p,
                       nq_blocks, nkv_blocks);
    if (launch_failed("bwd_reduce_kernel")) return BB_ERR_LAUNCH;
  }
  return BB_OK;
}

}  // namespace bb
