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
// wave) and, at small sizes, the longest slice: hence slices down to a single pair (fine_slice_f32).
// n = 1024, 2 heads: dQ 18 us, dK/dV 27 us, reduction 4 us, where one workgroup per block with vector
// arithmetic took 313 and 358; n = 4096, 24 slices, forward and backward: 0.73 ms against 10.7.
// (dK/dV is held to two waves per SIMD: 29 registers spilled, but 0.73 against 0.78 ms.)
#include "bwd_kernels.h"
#include "f32_ops.h"

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
  // gradients of a padded key are exactly 0 (selected, not multiplied: its K row may hold anything)
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

int launch_bwd_f32(const BwdParams& p, hipStream_t stream) {
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
