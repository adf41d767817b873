// Backward kernels, fp32 end to end.  Same calculus as the bf16 kernels (eq. (AT) of Sec. 2
// differentiated on the blocked pattern of App. D):
//   dV = P^T dO;  dP = dO V^T;  D_i = sum_c dO_ic O_ic;  dS = P o (dP - D);
//   dQ = scale dS K;  dK = scale dS^T Q,
// with P recomputed from Q, K and the forward's LSE.  No atomics: a work item is a slice of a query
// block's key-block list (dQ) or of a key block's query-block list (dK, dV); where a list has several
// slices, bwd_reduce_kernel adds their partial sums in slice order.
//
// fp32 MFMA 32x32x2 throughout, four waves per item, a wave per 32x32 quarter of every block pair
// (f32_ops.h).  What bounds them is the fp32 matrix rate (a block pair is 96 / 128 MFMAs of 64 cycles per
// wave) and, at small sizes, the longest slice: hence slices down to a single pair (fine_slice_f32), and for the
// smallest launches the kernels at the end of this file.
// n = 4096, 24 slices, forward and backward: 0.73 ms, where one workgroup per block with vector arithmetic took 10.7.
// (dK/dV is held to two waves per SIMD: 29 registers spilled, but 0.73 against 0.78 ms.)
#include "bwd_kernels.h"
#include "f32_ops.h"
#include "f32_rows.h"

#include <cstdio>

namespace bb {

namespace {

// [64 x 32] accumulator pair (rows d, column = this lane's sequence position) -> dst_row[d].
__device__ __forceinline__ void store_rows_f32(float* dst_row, const f32x16 (&a)[2], int hf) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = a[dt][r4 * 4 + e];
      *reinterpret_cast<f32x4*>(dst_row + dt * 32 + acc_row(r4 * 4, hf)) = v;
    }
}

// Accumulators of one wave to another through LDS, register by register (2048 floats).
__device__ __forceinline__ void hand_over(float* slot, int lane, const f32x16 (&a)[2]) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) slot[(dt * 16 + r) * 64 + lane] = a[dt][r];
}
__device__ __forceinline__ void take_over(const float* slot, int lane, f32x16 (&a)[2]) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[dt][r] += slot[(dt * 16 + r) * 64 + lane];
}

__device__ __forceinline__ void clear(f32x16 (&a)[2]) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[dt][r] = 0.f;
}

}  // namespace

// ---------------------------------------------------------------------------------------
// dQ (and the row sums D): one work item = (batch*head, query block, slice of its key-block list).
// Wave (qh, kh): 32 queries against 32 keys of every block; S^T, dP^T, dS^T are [keys x queries],
// dQ^T += K^T dS^T; the two key halves' shares are added in LDS.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreadsF32) void bwd_f32_dq_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(16))) float lds_k[kBlk * kF32Stride];
  __shared__ __attribute__((aligned(16))) float lds_v[kBlk * kF32Stride];
  __shared__ int klist[kChunkMax];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  WorkItem it;
  if (!decode_item(p.split, pat, p.BH, blockIdx.x, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int hf = lane >> 5, col = lane & 31;
  const int qh = wv & 1, kh = wv >> 1;
  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;
  const size_t qrow = bh_row0 + static_cast<size_t>(it.j) * kBlk + qh * 32 + col;
  const float* Kp = static_cast<const float*>(p.K);
  const float* Vp = static_cast<const float*>(p.V);

  f32x4 qf[8], gf[8];  // Q and dO rows of this lane's query, half of d each
  row_fragments_f32(static_cast<const float*>(p.Q) + qrow * kDim, hf, qf);
  row_fragments_f32(static_cast<const float*>(p.dO) + qrow * kDim, hf, gf);
  // a query block that was skipped (no valid position) behaves like rows without a valid key
  const bool skip = p.skip_q && key_valid_bits(p.kmask, bi, p.n, it.j) == 0;
  float dsum, lse2;
  {
    f32x4 of[8];
    row_fragments_f32(static_cast<const float*>(p.O) + qrow * kDim, hf, of);
    float part = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) part = __builtin_fmaf(gf[u][e], of[u][e], part);
    dsum = half_sum(part);
    if (skip) dsum = 0.f;
    const float lse = p.LSE[qrow];
    lse2 = (skip || lse == neg_inf()) ? __builtin_inff() : lse * kLog2e;  // no valid key: every P is 0
    if (it.chunk == 0 && kh == 0 && hf == 0) {
      p.Dvec[qrow] = dsum;
      p.Lvec[qrow] = lse2;
    }
  }
  const int cnt = skip ? 0 : build_key_list(pat, p.rand_idx, p.r, p.kmask, p.n, bi, h, it, klist);
  __syncthreads();

  const float c = p.c;
  // attention dropout: dP = M / (1 - p) o (dO V^T), M this row of the keep mask
  const uint32_t drop_rk = p.drop.thr ? drop_row_key(p.drop, static_cast<uint32_t>(qrow)) : 0u;
  f32x16 dq[2];
  clear(dq);
  f32x4 kreg[kVecPerThreadF32], vreg[kVecPerThreadF32];
  if (cnt > 0) {
    const size_t row0 = bh_row0 + static_cast<size_t>(klist[0]) * kBlk;
    tile_fetch_f32(Kp + row0 * kDim, kreg);
    tile_fetch_f32(Vp + row0 * kDim, vreg);
  }
  for (int i = 0; i < cnt; ++i) {
    const int kb = klist[i];
    __syncthreads();  // everyone is done reading the previous tiles
    tile_store_f32(lds_k, kreg);
    tile_store_f32(lds_v, vreg);
    __syncthreads();
    if (i + 1 < cnt) {
      const size_t row0 = bh_row0 + static_cast<size_t>(klist[i + 1]) * kBlk;
      tile_fetch_f32(Kp + row0 * kDim, kreg);
      tile_fetch_f32(Vp + row0 * kDim, vreg);
    }
    uint32_t valid = ~0u;  // bit acc_row(r, 0): this lane's r-th key
    if (p.kmask) valid = static_cast<uint32_t>(key_valid_bits(p.kmask, bi, p.n, kb) >> (kh * 32)) >> (hf * 4);

    f32x16 s, dp;
    mfma_rows_f32(lds_k + (kh * 32 + col) * kF32Stride, hf, qf, s);
    mfma_rows_f32(lds_v + (kh * 32 + col) * kF32Stride, hf, gf, dp);
    if (p.drop.thr) {
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const uint32_t key = static_cast<uint32_t>(kb * kBlk + kh * 32 + acc_row(r, hf));
        const uint32_t wd = drop_word(drop_rk, key >> 1);
        dp[r] = drop_keep_even(wd, p.drop.thr) ? dp[r] * p.drop.rs : 0.f;
        dp[r + 1] = drop_keep_odd(wd, p.drop.thr) ? dp[r + 1] * p.drop.rs : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float ds = fast_exp2(__builtin_fmaf(s[r], c, -lse2)) * (dp[r] - dsum);
      s[r] = (valid >> acc_row(r, 0)) & 1 ? ds : 0.f;
    }
    mfma_columns_f32(lds_k + kh * 32 * kF32Stride, hf, col, s, dq);
  }

  __syncthreads();  // the tiles are no longer read
  float* const slot = lds_k + qh * (32 * 64);
  if (kh == 1) hand_over(slot, lane, dq);
  __syncthreads();
  if (kh == 1) return;
  take_over(slot, lane, dq);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[dt][r] *= p.scale;
  if (it.nchunks == 1)
    store_rows_f32(p.dQ + qrow * kDim, dq, hf);
  else
    store_rows_f32(p.part_dq + static_cast<size_t>(it.slot) * (kBlk * kDim) + (qh * 32 + col) * kDim, dq, hf);
}

// ---------------------------------------------------------------------------------------
// dK, dV: one work item = (batch*head, key block k, slice of its query-block list).  Slice u of ns takes
// entries u, u + ns, ... of the list (a non-global key block's list can be of any length: the rows of
// rand_idx that name it).  Wave (qh, kh): 32 queries against 32 keys, S, dP, dS are [queries x keys],
// dV^T += dO^T P and dK^T += Q^T dS; the two query halves' shares are added in LDS.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreadsF32) __attribute__((amdgpu_waves_per_eu(2))) void bwd_f32_dkv_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(16))) float lds_q[kBlk * kF32Stride];
  __shared__ __attribute__((aligned(16))) float lds_do[kBlk * kF32Stride];
  __shared__ __attribute__((aligned(16))) float lds_lse[kBlk], lds_d[kBlk];
  __shared__ int jlist[kMaxBwdBlocks];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  KeyItem it;
  if (!decode_key_item(p, pat, blockIdx.x, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int hf = lane >> 5, col = lane & 31;
  const int qh = wv & 1, kh = wv >> 1;
  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;
  const size_t krow = bh_row0 + static_cast<size_t>(it.k) * kBlk + kh * 32 + col;
  const float* Qp = static_cast<const float*>(p.Q);
  const float* Gp = static_cast<const float*>(p.dO);

  f32x4 kf[8], vf[8];
  row_fragments_f32(static_cast<const float*>(p.K) + krow * kDim, hf, kf);
  row_fragments_f32(static_cast<const float*>(p.V) + krow * kDim, hf, vf);
  const bool key_valid = !p.kmask || p.kmask[static_cast<size_t>(bi) * p.n + it.k * kBlk + kh * 32 + col] != 0;
  const int total = build_query_list(p, pat, bi, h, it.k, jlist, wv == 0);
  __syncthreads();

  const float c = p.c;
  f32x16 dk[2], dv[2];
  clear(dk);
  clear(dv);
  f32x4 qreg[kVecPerThreadF32], greg[kVecPerThreadF32];
  float lreg = 0.f;  // threads 0 .. 63: LSE of row tid of the list entry, 64 .. 127: D
  auto fetch = [&](int u) {
    const size_t row0 = bh_row0 + static_cast<size_t>(jlist[u]) * kBlk;
    tile_fetch_f32(Qp + row0 * kDim, qreg);
    tile_fetch_f32(Gp + row0 * kDim, greg);
    if (wv < 2) lreg = (wv == 0 ? p.Lvec : p.Dvec)[row0 + lane];
  };
  if (it.chunk < total) fetch(it.chunk);
  for (int u = it.chunk; u < total; u += it.nchunks) {
    const int j = jlist[u];
    __syncthreads();  // everyone is done reading the previous tiles
    tile_store_f32(lds_q, qreg);
    tile_store_f32(lds_do, greg);
    if (wv < 2) (wv == 0 ? lds_lse : lds_d)[lane] = lreg;
    __syncthreads();
    if (u + it.nchunks < total) fetch(u + it.nchunks);

    f32x16 s, dp;
    mfma_rows_f32(lds_q + (qh * 32 + col) * kF32Stride, hf, kf, s);
    mfma_rows_f32(lds_do + (qh * 32 + col) * kF32Stride, hf, vf, dp);
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(lds_lse + qh * 32 + acc_row(r4 * 4, hf));
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(lds_d + qh * 32 + acc_row(r4 * 4, hf));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = r4 * 4 + e;
        const float pr = fast_exp2(__builtin_fmaf(s[r], c, -l4[e]));
        // attention dropout: dV takes the kept, rescaled probabilities; dP is masked the same way
        float mr = 1.f;
        if (p.drop.thr)
          mr = drop_keep(p.drop, static_cast<uint32_t>(bh_row0 + j * kBlk + qh * 32 + acc_row(r, hf)),
                         static_cast<uint32_t>(it.k * kBlk + kh * 32 + col))
                   ? p.drop.rs : 0.f;
        s[r] = pr * mr;
        dp[r] = pr * (dp[r] * mr - d4[e]);
      }
    }
    mfma_columns_f32(lds_do + qh * 32 * kF32Stride, hf, col, s, dv);
    mfma_columns_f32(lds_q + qh * 32 * kF32Stride, hf, col, dp, dk);
  }

  __syncthreads();  // the tiles are no longer read
  if (qh == 1) {
    hand_over(lds_q + kh * (32 * 64), lane, dk);
    hand_over(lds_do + kh * (32 * 64), lane, dv);
  }
  __syncthreads();
  if (qh == 1) return;
  take_over(lds_q + kh * (32 * 64), lane, dk);
  take_over(lds_do + kh * (32 * 64), lane, dv);
  // gradients of a padded key are exactly 0 (selected, not multiplied: what was summed for it may be anything)
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      dk[dt][r] = key_valid ? dk[dt][r] * p.scale : 0.f;
      dv[dt][r] = key_valid ? dv[dt][r] : 0.f;
    }
  const size_t off = it.nchunks == 1 ? krow * kDim
                                     : static_cast<size_t>(it.slot) * (kBlk * kDim) + (kh * 32 + col) * kDim;
  store_rows_f32((it.nchunks == 1 ? p.dK : p.part_dk) + off, dk, hf);
  store_rows_f32((it.nchunks == 1 ? p.dV : p.part_dv) + off, dv, hf);
}

// ---------------------------------------------------------------------------------------
// Small launches (rows_f32_bwd): a workgroup per eight queries (dQ) or eight keys (dK, dV), see f32_rows.h.  Tiles come
// as a stream of quarters (sixteen rows of both), one ahead.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kRowsThreadsF32) __attribute__((amdgpu_waves_per_eu(2))) void bwd_rows_f32_dq_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char ring_all[kRowsWavesF32][2][2][kQuarterF32];  // a wave's K and V quarters; then its dQ
  __shared__ int klist_all[kRowsWavesF32][kMaxListLen];
  __shared__ uint32_t key_bits_all[kRowsWavesF32][kMaxListLen][2];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  OwnItem it;
  if (!decode_own(pat, p.BH, blockIdx.x, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowsLane l(lane);
  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;
  const size_t row0 = bh_row0 + static_cast<size_t>(it.j) * kBlk + it.first;
  const float* Kp = static_cast<const float*>(p.K) + bh_row0 * kDim;
  const float* Vp = static_cast<const float*>(p.V) + bh_row0 * kDim;

  f32x4 qf[2][4], gf[2][4];
  own_rows(static_cast<const float*>(p.Q) + row0 * kDim, l, qf);
  own_rows(static_cast<const float*>(p.dO) + row0 * kDim, l, gf);
  float dsum[2], lse2[2];
  {
    f32x4 of[2][4];
    own_rows(static_cast<const float*>(p.O) + row0 * kDim, l, of);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float part = 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) part = __builtin_fmaf(gf[q][u][e], of[q][u][e], part);
      dsum[q] = part;
      lse2[q] = p.LSE[row0 + 4 * q + l.t];
    }
  }
  // a query block that was skipped (no valid position) behaves like rows without a valid key
  const bool skip = p.skip_q && !block_any_valid_scalar(p.kmask, bi, p.n, it.j);
  int cnt = 0;
  KeyList list = {0, 0, 0u};
  if (!skip) {
    list = own_key_list(pat, p.rand_idx, p.r, p.kmask, p.n, bi, h, it, wv, lane, klist_all[wv], key_bits_all[wv]);
    cnt = __builtin_amdgcn_readfirstlane(list.cnt);
  }
  uint32_t drop_rk[2] = {0u, 0u};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    dsum[q] = skip ? 0.f : add_over_groups(dsum[q]);
    lse2[q] = (skip || lse2[q] == neg_inf()) ? __builtin_inff() : lse2[q] * kLog2e;  // no valid key: every P is 0
    if (wv == 0 && lane < 4) {
      p.Dvec[row0 + 4 * q + lane] = dsum[q];
      p.Lvec[row0 + 4 * q + lane] = lse2[q];
    }
    if (p.drop.thr) drop_rk[q] = drop_row_key(p.drop, static_cast<uint32_t>(row0 + 4 * q + l.t));
  }

  const float c = p.c;
  f32x4 dq[2][4];
  clear_own(dq);
  const QuarterLoads ql(lane);
  const QuarterForms qforms(l);
  const unsigned ring_a = lds_addr(ring_all[wv]);
  // quarters of the list's K and V tiles, one ahead
  auto request = [&](int i, int kt) {
    const size_t off = static_cast<size_t>(__builtin_amdgcn_readlane(list.entry, i)) * (kBlk * kDim) + kt * 16 * kDim;
    ql.request(Kp + off, ring_a + (kt & 1) * (2 * kQuarterF32));
    ql.request(Vp + off, ring_a + (kt & 1) * (2 * kQuarterF32) + kQuarterF32);
  };
  if (cnt > 0) request(0, 0);
  for (int i = 0; i < cnt; ++i) {
    const int kb = __builtin_amdgcn_readlane(list.entry, i);
    const bool cut = (list.partial >> i) & 1;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      wait_lds_reads();  // the other place of the ring is free
      if (kt < 3 || i + 1 < cnt) {
        request(kt < 3 ? i : i + 1, (kt + 1) & 3);
        wait_tile_loads<2 * kQuarterLoads>();
      } else {
        wait_tile_loads<0>();
      }
      const char (*quarter)[kQuarterF32] = ring_all[wv][kt & 1];
      f32x4 x[4], y[4];
      float s[2], dp[2];
      qforms.row_form(quarter[0], x);
      qforms.row_form(quarter[1], y);
      row_products(x, qf, s, y, gf, dp);
      const uint32_t key = static_cast<uint32_t>(kb * kBlk + l.row(kt));
      const bool valid = !cut || row_valid(key_bits_all[wv][i], l, kt);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (p.drop.thr) {  // dP = M / (1 - p) o (dO V^T), M the keep mask
          const uint32_t wd = drop_word(drop_rk[q], key >> 1);
          dp[q] = ((key & 1u) ? drop_keep_odd(wd, p.drop.thr) : drop_keep_even(wd, p.drop.thr)) ? dp[q] * p.drop.rs : 0.f;
        }
        const float ds = fast_exp2(__builtin_fmaf(s[q], c, -lse2[q])) * (dp[q] - dsum[q]);
        s[q] = valid ? ds : 0.f;  // (its K row is multiplied by this 0 below, and has to be finite)
      }
      qforms.column_form(quarter[0], x);
      add_rows(x, s, dq);
    }
  }

  wait_lds_reads();
  auto dq_of = [&](int v) { return reinterpret_cast<float (*)[kDim]>(ring_all[v][0][0]); };
  store_own(dq_of(wv), l, dq);
  __syncthreads();
  float acc = 0.f;
#pragma unroll
  for (int v = 0; v < kRowsWavesF32; ++v) acc += dq_of(v)[wv][lane];
  p.dQ[(row0 + wv) * kDim + lane] = acc * p.scale;
}

// Query blocks that attend key block k, one in kRowsWavesF32 of them (those of wave wv) into jlist, by that wave; returns how many.
// A lane looks at query block j0 + lane: one trip to memory for up to four random blocks a row.
__device__ __forceinline__ int own_query_list(const BwdParams& p, const Pattern& pat, int bi, int h, int k, bool key_global,
                                              int wv, int lane, int* jlist) {
  const int32_t* tbl = p.rand_idx ? p.rand_idx + static_cast<size_t>(h) * p.nb * p.r : nullptr;
  int cnt = 0;
  for (int j0 = 0; j0 < p.nb; j0 += 64) {
    const int j = j0 + lane;
    bool valid = j < p.nb;
    if (valid && !key_global && !pat.is_global(j) && !pat.in_window(j, k)) {
      valid = false;
      for (int t0 = 0; tbl && t0 < p.r; t0 += 4) {
        int e[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) e[t] = tbl[static_cast<size_t>(j) * p.r + (t0 + t < p.r ? t0 + t : p.r - 1)];
#pragma unroll
        for (int t = 0; t < 4; ++t) valid |= e[t] == k;
      }
    }
    if (p.skip_q && valid) valid = block_has_valid_key(p.kmask, bi, p.n, j);
    const uint64_t mask = __ballot(valid);
    const int rank = cnt + mask_rank(mask);
    if (valid && rank % kRowsWavesF32 == wv) jlist[rank / kRowsWavesF32] = j;
    cnt += static_cast<int>(__popcll(mask));
  }
  asm volatile("" ::: "memory");  // the same wave reads the list: LDS keeps a wave's accesses in order, the compiler must too
  return cnt > wv ? (cnt - wv + kRowsWavesF32 - 1) / kRowsWavesF32 : 0;
}

__global__ __launch_bounds__(kRowsThreadsF32) __attribute__((amdgpu_waves_per_eu(2))) void bwd_rows_f32_dkv_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char ring_all[kRowsWavesF32][2][2][kQuarterF32];  // a wave's Q and dO quarters; then its dK, dV
  __shared__ __attribute__((aligned(256))) float vec_all[kRowsWavesF32][2][2][kBlk];          // LSE log2(e) and D of the rows of an entry
  __shared__ int jlist_all[kRowsWavesF32][kMaxListLen];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  OwnItem it;
  if (!decode_own(pat, p.BH, blockIdx.x, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowsLane l(lane);
  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;
  const size_t key0 = bh_row0 + static_cast<size_t>(it.j) * kBlk + it.first;  // first own key
  const float* Qp = static_cast<const float*>(p.Q) + bh_row0 * kDim;
  const float* Gp = static_cast<const float*>(p.dO) + bh_row0 * kDim;

  f32x4 kf[2][4], vf[2][4];
  own_rows(static_cast<const float*>(p.K) + key0 * kDim, l, kf);
  own_rows(static_cast<const float*>(p.V) + key0 * kDim, l, vf);
  const int cnt = __builtin_amdgcn_readfirstlane(own_query_list(p, pat, bi, h, it.j, it.global, wv, lane, jlist_all[wv]));

  const float c = p.c;
  f32x4 dk[2][4], dv[2][4];
  clear_own(dk);
  clear_own(dv);
  const QuarterLoads ql(lane);
  const QuarterForms qforms(l);
  const unsigned ring_a = __builtin_amdgcn_readfirstlane(lds_addr(ring_all[wv]));
  const unsigned vec_a = __builtin_amdgcn_readfirstlane(lds_addr(vec_all[wv]));
  // quarters of the list's Q and dO tiles, one ahead; LSE and D of an entry come with its first
  auto entry = [&](int i) { return __builtin_amdgcn_readfirstlane(jlist_all[wv][i]); };
  auto request = [&](int i, int j, int kt) {
    const size_t off = static_cast<size_t>(j) * (kBlk * kDim) + kt * 16 * kDim;
    ql.request(Qp + off, ring_a + (kt & 1) * (2 * kQuarterF32));
    ql.request(Gp + off, ring_a + (kt & 1) * (2 * kQuarterF32) + kQuarterF32);
    if (kt == 0) {
      const size_t row = bh_row0 + static_cast<size_t>(j) * kBlk;
      vec_load_async(p.Lvec + row, vec_a + (i & 1) * (2 * kBlk * 4), lane);
      vec_load_async(p.Dvec + row, vec_a + (i & 1) * (2 * kBlk * 4) + kBlk * 4, lane);
    }
  };
  if (cnt > 0) request(0, entry(0), 0);
  for (int i = 0; i < cnt; ++i) {
    const int j = entry(i);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      wait_lds_reads();  // the other place of the ring is free
      if (kt < 3) {
        request(i, j, kt + 1);
        wait_tile_loads<2 * kQuarterLoads>();
      } else if (i + 1 < cnt) {
        request(i + 1, entry(i + 1), 0);
        wait_tile_loads<2 * kQuarterLoads + 2>();
      } else {
        wait_tile_loads<0>();
      }
      const char (*quarter)[kQuarterF32] = ring_all[wv][kt & 1];
      f32x4 x[4], y[4];
      float s[2], dp[2];
      qforms.row_form(quarter[0], x);
      qforms.row_form(quarter[1], y);
      row_products(x, kf, s, y, vf, dp);
      const float lse2 = vec_all[wv][i & 1][0][l.row(kt)], dsum = vec_all[wv][i & 1][1][l.row(kt)];
      const uint32_t rk = p.drop.thr ? drop_row_key(p.drop, static_cast<uint32_t>(bh_row0 + static_cast<size_t>(j) * kBlk + l.row(kt))) : 0u;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float pr = fast_exp2(__builtin_fmaf(s[q], c, -lse2));
        float mr = 1.f;  // attention dropout: dV takes the kept, rescaled probabilities; dP is masked the same way
        if (p.drop.thr) {
          const uint32_t key = static_cast<uint32_t>(it.j * kBlk + it.first + 4 * q + l.t);
          const uint32_t wd = drop_word(rk, key >> 1);
          mr = ((key & 1u) ? drop_keep_odd(wd, p.drop.thr) : drop_keep_even(wd, p.drop.thr)) ? p.drop.rs : 0.f;
        }
        s[q] = pr * mr;
        dp[q] = pr * (dp[q] * mr - dsum);
      }
      qforms.column_form(quarter[1], y);
      qforms.column_form(quarter[0], x);
      add_rows(y, s, dv);
      add_rows(x, dp, dk);
    }
  }

  wait_lds_reads();
  auto dk_of = [&](int v) { return reinterpret_cast<float (*)[kDim]>(ring_all[v][0][0]); };
  auto dv_of = [&](int v) { return reinterpret_cast<float (*)[kDim]>(ring_all[v][0][1]); };
  store_own(dk_of(wv), l, dk);
  store_own(dv_of(wv), l, dv);
  const bool key_valid = !p.kmask || p.kmask[static_cast<size_t>(bi) * p.n + it.j * kBlk + it.first + wv] != 0;
  __syncthreads();
  float a = 0.f, b = 0.f;
#pragma unroll
  for (int v = 0; v < kRowsWavesF32; ++v) {
    a += dk_of(v)[wv][lane];
    b += dv_of(v)[wv][lane];
  }
  // gradients of a padded key are exactly 0 (selected, not multiplied: what was summed for it may be anything)
  p.dK[(key0 + wv) * kDim + lane] = key_valid ? a * p.scale : 0.f;
  p.dV[(key0 + wv) * kDim + lane] = key_valid ? b : 0.f;
}

int launch_bwd_f32(const BwdParams& p, hipStream_t stream) {
  if (rows_f32_bwd(p.BH, p.nb)) {
    const unsigned grid = own_grid(p.BH, p.nb);
    hipLaunchKernelGGL(bwd_rows_f32_dq_kernel, dim3(grid), dim3(kRowsThreadsF32), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
      hipLaunchKernelGGL(bwd_rows_f32_dkv_kernel, dim3(grid), dim3(kRowsThreadsF32), 0, stream, p);
      e = hipGetLastError();
    }
    if (e != hipSuccess) {
      fprintf(stderr, "bigbird: launch of the fp32 backward kernels failed: %s\n", hipGetErrorString(e));
      return BB_ERR_LAUNCH;
    }
    return BB_OK;
  }
  const unsigned qgrid = DieItems(p.BH, p.split.items_per_bh).grid();
  const unsigned kvgrid = DieItems(p.BH, p.kv.items_per_bh).grid();
  hipLaunchKernelGGL(bwd_f32_dq_kernel, dim3(qgrid), dim3(kThreadsF32), 0, stream, p);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(bwd_f32_dkv_kernel, dim3(kvgrid), dim3(kThreadsF32), 0, stream, p);
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    fprintf(stderr, "bigbird: launch of the fp32 backward kernels failed: %s\n", hipGetErrorString(e));
    return BB_ERR_LAUNCH;
  }
  return launch_bwd_reduce(p, stream);
}

}  // namespace bb
