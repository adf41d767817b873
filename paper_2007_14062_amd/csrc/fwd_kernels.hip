// Forward kernels: the fp32 fused kernel (S^T = K Q^T -> online softmax ->
// O^T += V^T P^T per query block and slice of its key-block list), the merge of
// sliced rows, and the launch logic.  The bf16 fused kernel is in fwd_bf16.hip.
//
// Eq. (AT) of Sec. 2 per head on the blocked pattern of App. D.  Each block pair
// is a dense 64x64x64 contraction, which is what the MFMA units are for.  The
// scores are produced transposed (keys along MFMA rows, queries along MFMA
// columns) so that one lane owns one query column: the row maximum and row sum of
// the softmax are in-lane reductions plus one exchange between the two 32-lane
// halves, and the probabilities sit in registers exactly where the second MFMA
// wants its B operand (the contraction order over keys is free, so V^T is read
// from LDS in the matching permuted key order).
#include "f32_ops.h"
#include "f32_rows.h"
#include "fwd_epilogue.h"

#include <cstdio>

namespace bb {

// fp32 end to end: fp32 MFMA 32x32x2.  Four waves per work item; wave (qh, kh) takes 32 queries against
// 32 of the 64 keys of every block with an online softmax of its own, and the two key halves are merged
// in LDS at the end.  What bounds it is the fp32 matrix rate (a block pair is 64 MFMAs of 64 cycles per
// wave: 2 us) and, at small sizes, the length of the longest slice: hence the fine slices
// (fine_slice_f32).  n = 2048, 12 heads: 50 us a call, where two waves over slices of 8 blocks took 92.  The smallest
// launches take fwd_rows_f32.
__global__ __launch_bounds__(kThreadsF32) void fwd_kernel_f32(FwdParams p) {
  __shared__ __attribute__((aligned(16))) float lds_k[kBlk * kF32Stride];
  __shared__ __attribute__((aligned(16))) float lds_v[kBlk * kF32Stride];
  __shared__ float mrg_m[kBlk], mrg_l[kBlk];
  __shared__ int klist[kChunkMax];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  WorkItem it;
  if (!decode_item(p.split, pat, p.BH, blockIdx.x, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int hf = lane >> 5, col = lane & 31;
  const int qh = wv & 1, kh = wv >> 1;

  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;    // first row of this (batch, head)
  const size_t qrow = bh_row0 + it.j * kBlk + qh * 32 + col;  // this lane's query row
  const float* Kp = static_cast<const float*>(p.K);
  const float* Vp = static_cast<const float*>(p.V);

  // Q^T operand: MFMA contraction slot hf of step (u, e) is d = 8u + 4hf + e.
  f32x4 qf[8];
  row_fragments_f32(static_cast<const float*>(p.Q) + qrow * kDim, hf, qf);

  // (a query block without a valid position, if the caller asked for those to be skipped, is an
  // empty row: O = 0, LSE = -inf through the usual end of an item)
  const bool skip = p.skip_q && key_valid_bits(p.kmask, bi, p.n, it.j) == 0;
  const int cnt = skip ? 0 : build_key_list(pat, p.rand_idx, p.r, p.kmask, p.n, bi, h, it, klist);
  __syncthreads();

  f32x16 o[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  // attention dropout: the key of this lane's row of the keep mask
  const uint32_t drop_rk = p.drop.thr ? drop_row_key(p.drop, static_cast<uint32_t>(qrow)) : 0u;
  float m_run = neg_inf();  // running maximum of the raw scores q.k (both lane halves agree)
  float l_run = 0.f;        // this lane's share of the running sum of 2^((q.k - m) c)
  const float c = p.c;

  f32x4 kreg[kVecPerThreadF32], vreg[kVecPerThreadF32];
  if (cnt > 0) {
    const size_t krow0 = bh_row0 + static_cast<size_t>(klist[0]) * kBlk;
    tile_fetch_f32(Kp + krow0 * kDim, kreg);
    tile_fetch_f32(Vp + krow0 * kDim, vreg);
  }

  for (int i = 0; i < cnt; ++i) {
    const int kb = klist[i];
    __syncthreads();  // everyone is done reading the previous tiles
    tile_store_f32(lds_k, kreg);
    tile_store_f32(lds_v, vreg);
    __syncthreads();
    if (i + 1 < cnt) {
      const size_t krow0 = bh_row0 + static_cast<size_t>(klist[i + 1]) * kBlk;
      tile_fetch_f32(Kp + krow0 * kDim, kreg);
      tile_fetch_f32(Vp + krow0 * kDim, vreg);
    }
    uint64_t vbits = ~0ull;
    if (p.kmask) vbits = key_valid_bits(p.kmask, bi, p.n, kb);

    // ---- S^T: rows = this wave's 32 keys, columns = its 32 queries
    f32x16 s;
    mfma_rows_f32(lds_k + (kh * 32 + col) * kF32Stride, hf, qf, s);

    // ---- padded keys -> -inf (only blocks that are partly padded take this path)
    if (vbits != ~0ull) {
      const uint32_t mine = static_cast<uint32_t>(vbits >> (kh * 32)) >> (hf * 4);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (!((mine >> acc_row(r, 0)) & 1)) s[r] = neg_inf();
    }

    // ---- online softmax (base 2, scale folded into c)
    float mloc = neg_inf();
#pragma unroll
    for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[r]);
    mloc = half_max(mloc);
    const float m_new = fmaxf(m_run, mloc);
    const float m_use = (m_new == neg_inf()) ? 0.f : m_new;
    const float alpha = fast_exp2((m_run - m_use) * c);
    const float mc = m_use * c;
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float pv = fast_exp2(__builtin_fmaf(s[r], c, -mc));
      s[r] = pv;
      lsum += pv;
    }
    l_run = l_run * alpha + lsum;
    m_run = m_new;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;

    // ---- attention dropout: the row sums above are those of the undropped probabilities; what
    // multiplies V is the kept part (registers r, r+1 are keys 2m, 2m+1: one word of the mask)
    if (p.drop.thr) {
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const uint32_t key = static_cast<uint32_t>(kb * kBlk + kh * 32 + acc_row(r, hf));
        const uint32_t wd = drop_word(drop_rk, key >> 1);
        if (!drop_keep_even(wd, p.drop.thr)) s[r] = 0.f;
        if (!drop_keep_odd(wd, p.drop.thr)) s[r + 1] = 0.f;
      }
    }

    // ---- O^T += V^T P^T: the S^T accumulator is the B operand as it stands
    mfma_columns_f32(lds_v + kh * 32 * kF32Stride, hf, col, s, o);
  }

  // ---- merge the two key halves: waves kh = 1 hand over, waves kh = 0 finish
  float l_tot = half_sum(l_run);
  __syncthreads();  // the tiles are no longer read
  float* const slot = lds_k + qh * (32 * 64);
  if (kh == 1) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) slot[(dt * 16 + r) * 64 + lane] = o[dt][r];
    if (hf == 0) {
      mrg_m[qh * 32 + col] = m_run;
      mrg_l[qh * 32 + col] = l_tot;
    }
  }
  __syncthreads();
  if (kh == 1) return;
  const float m1 = mrg_m[qh * 32 + col], l1 = mrg_l[qh * 32 + col];
  const float m_all = fmaxf(m_run, m1);
  const float m_ref = m_all == neg_inf() ? 0.f : m_all;
  const float w0 = fast_exp2((m_run - m_ref) * c), w1 = fast_exp2((m1 - m_ref) * c);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = o[dt][r] * w0 + slot[(dt * 16 + r) * 64 + lane] * w1;
  l_tot = l_tot * w0 + l1 * w1;
  fwd_store(p, it, o, m_all, l_tot, c, qrow, qh * 32 + col, hf);
}

// Small fp32 launches (rows_f32_fwd): a workgroup per eight queries (f32_rows.h), an online softmax per wave over its share
// of the key blocks, the waves merged in LDS: one launch.  (K and V as one stream of quarters through a ring, three
// ahead, took 12.1 us where this takes 11.7: 2 slices of n = 1024.)
__global__ __launch_bounds__(kRowsThreadsF32) __attribute__((amdgpu_waves_per_eu(2))) void fwd_rows_f32(FwdParams p) {
  __shared__ __attribute__((aligned(1024))) char k_all[kRowsWavesF32][4][kQuarterF32];  // a wave's K tile; then its O
  __shared__ float m_all[kRowsWavesF32][kOwn], l_all[kRowsWavesF32][kOwn];
  __shared__ int klist_all[kRowsWavesF32][kMaxListLen];
  __shared__ uint32_t key_bits_all[kRowsWavesF32][kMaxListLen][2];

  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  OwnItem it;
  if (!decode_own(pat, p.BH, blockIdx.x, &it)) return;
  const int bi = it.bh / p.H, h = it.bh % p.H;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowsLane l(lane);
  const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;
  const size_t row0 = bh_row0 + static_cast<size_t>(it.j) * kBlk + it.first;  // first own query
  const float* Kp = static_cast<const float*>(p.K) + bh_row0 * kDim;
  const float* Vp = static_cast<const float*>(p.V) + bh_row0 * kDim;

  f32x4 qf[2][4];
  own_rows(static_cast<const float*>(p.Q) + row0 * kDim, l, qf);
  // (a query block without a valid position, if the caller asked for those to be skipped, is an empty row)
  const bool skip = p.skip_q && !block_any_valid_scalar(p.kmask, bi, p.n, it.j);
  int cnt = 0;
  KeyList list = {0, 0, 0u};
  if (!skip) {
    list = own_key_list(pat, p.rand_idx, p.r, p.kmask, p.n, bi, h, it, wv, lane, klist_all[wv], key_bits_all[wv]);
    cnt = __builtin_amdgcn_readfirstlane(list.cnt);
  }

  const float c = p.c;
  f32x4 o[2][4];
  clear_own(o);
  float m_run[2] = {neg_inf(), neg_inf()};  // running maxima of the raw scores of queries 4 q + t
  float l_run[2] = {0.f, 0.f};              // this lane's share of the sums of 2^((q.k - m) c)
  uint32_t drop_rk[2] = {0u, 0u};
  if (p.drop.thr) {
#pragma unroll
    for (int q = 0; q < 2; ++q) drop_rk[q] = drop_row_key(p.drop, static_cast<uint32_t>(row0 + 4 * q + l.t));
  }
  // K goes through LDS, V straight to registers in the form its product wants; both are requested while the entry
  // before is in work
  const QuarterLoads ql(lane);
  const QuarterForms qforms(l);
  const unsigned k_a = lds_addr(k_all[wv]);
  f32x4 z[4][4];
  auto request_k = [&](int i) {
    const float* t = Kp + static_cast<size_t>(__builtin_amdgcn_readlane(list.entry, i)) * (kBlk * kDim);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) ql.request(t + kt * 16 * kDim, k_a + kt * kQuarterF32);
  };
  auto request_v = [&](int i, int kt) {
    const float* t = Vp + static_cast<size_t>(__builtin_amdgcn_readlane(list.entry, i)) * (kBlk * kDim);
#pragma unroll
    for (int s = 0; s < 4; ++s) z[kt][s] = *reinterpret_cast<const f32x4*>(t + (16 * kt + 4 * s + l.g) * kDim + 4 * l.m);
  };
  if (cnt > 0) {
    request_k(0);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) request_v(0, kt);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int i = 0; i < cnt; ++i) {
    const int kb = __builtin_amdgcn_readlane(list.entry, i);
    float s[4][2];
    wait_tile_loads<16 + 2 * kQuarterLoads>();  // half of K(i): the sixteen loads of V(i) are younger
#pragma unroll
    for (int kt = 0; kt < 4; kt += 2) {
      if (kt == 2) wait_tile_loads<16>();
      f32x4 x0[4], x1[4];
      qforms.row_form(k_all[wv][kt], x0);
      qforms.row_form(k_all[wv][kt + 1], x1);
      row_products(x0, qf, s[kt], x1, qf, s[kt + 1]);
    }
    wait_lds_reads();
    const bool more = i + 1 < cnt;
    if (more) request_k(i + 1);
    if ((list.partial >> i) & 1) {  // padded keys -> -inf (selected: their scores may be anything)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const bool valid = row_valid(key_bits_all[wv][i], l, kt);
#pragma unroll
        for (int q = 0; q < 2; ++q) s[kt][q] = valid ? s[kt][q] : neg_inf();
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float m_new = fmaxf(m_run[q], max_over_rows(fmaxf(fmaxf(s[0][q], s[1][q]), fmaxf(s[2][q], s[3][q]))));
      const float m_use = m_new == neg_inf() ? 0.f : m_new;
      const float alpha = fast_exp2((m_run[q] - m_use) * c);
      const float mc = m_use * c;
      float sum = 0.f;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        s[kt][q] = fast_exp2(__builtin_fmaf(s[kt][q], c, -mc));
        sum += s[kt][q];
      }
      l_run[q] = l_run[q] * alpha + sum;
      m_run[q] = m_new;
      const float al[4] = {of_position<0>(alpha), of_position<1>(alpha), of_position<2>(alpha), of_position<3>(alpha)};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int u = 0; u < 4; ++u) o[q][e][u] *= al[u];
    }
    if (p.drop.thr) {  // (the sums are those of the undropped probabilities)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const uint32_t key = static_cast<uint32_t>(kb * kBlk + l.row(kt));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t wd = drop_word(drop_rk[q], key >> 1);
          if (!((key & 1u) ? drop_keep_odd(wd, p.drop.thr) : drop_keep_even(wd, p.drop.thr))) s[kt][q] = 0.f;
        }
      }
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      add_rows(z[kt], s[kt], o);
      if (more) request_v(i + 1, kt);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  auto o_of = [&](int v) { return reinterpret_cast<float (*)[kDim]>(k_all[v][0]); };
  store_own(o_of(wv), l, o);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float sum = add_over_rows(l_run[q]);
    if (lane < 4) {
      m_all[wv][4 * q + lane] = m_run[q];
      l_all[wv][4 * q + lane] = sum;
    }
  }
  __syncthreads();
  // wave wv finishes query wv, lane d
  float M = neg_inf();
#pragma unroll
  for (int v = 0; v < kRowsWavesF32; ++v) M = fmaxf(M, m_all[v][wv]);
  const float ref = M == neg_inf() ? 0.f : M;
  float L = 0.f, acc = 0.f;
#pragma unroll
  for (int v = 0; v < kRowsWavesF32; ++v) {
    const float wgt = fast_exp2((m_all[v][wv] - ref) * c);  // 0 for a wave without a key
    L += l_all[v][wv] * wgt;
    acc += o_of(v)[wv][lane] * wgt;
  }
  static_cast<float*>(p.O)[(row0 + wv) * kDim + lane] = acc * (L > 0.f ? p.drop.rs / L : 0.f);  // (rs: 1, or the dropout scale)
  if (lane == 0) p.LSE[row0 + wv] = L > 0.f ? (M * c + fast_log2(L)) * kLn2 : neg_inf();
}

// Merge the slices of a split row: M = max m_c, L = sum l_c 2^(m_c - M),
// O = sum O~_c 2^(m_c - M) / L, LSE = (M + log2 L) ln 2.  Four workgroups per
// (batch, head, split row), 16 queries each; thread t owns 4 d columns of query
// t/16, so a wavefront reads four full 256-byte rows of every partial.
constexpr int kCombineThreads = 256;
constexpr int kCombineSplit = 4;  // workgroups per 64-query block

template <bool BF16>
__global__ __launch_bounds__(kCombineThreads) void fwd_combine_kernel(FwdParams p) {
  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  const int rows_per_bh = p.cmb_g_rows + p.cmb_s_rows;
  const int part = blockIdx.x % kCombineSplit;
  const int rowid = blockIdx.x / kCombineSplit;
  const int bh = rowid / rows_per_bh, rr = rowid % rows_per_bh;
  int j, nchunks, slot0;
  if (rr < p.cmb_g_rows) {
    j = pat.global_block(rr);
    nchunks = p.cmb_g_n;
    slot0 = bh * p.slots_per_bh + rr * p.cmb_g_n;
  } else {
    const int t = rr - p.cmb_g_rows;
    j = pat.sparse_block(t);
    nchunks = p.cmb_s_n;
    slot0 = bh * p.slots_per_bh + p.cmb_g_rows * p.cmb_g_n + t * p.cmb_s_n;
  }
  const int q = part * 16 + (threadIdx.x >> 4), d0 = (threadIdx.x & 15) * 4;
  const float* ml = p.part_ml + static_cast<size_t>(slot0) * (2 * kBlk) + q;
  const float* po = p.part_o + static_cast<size_t>(slot0) * (kBlk * kDim) + q * kDim + d0;
  // One pass with a running maximum, eight partials and their (m, l) requested together: a trip to
  // memory per eight slices, not one per slice.
  float M = neg_inf(), L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 8;
  for (int c0 = 0; c0 < nchunks; c0 += U) {
    f32x4 v[U];
    float mc[U], lc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cidx = c0 + u < nchunks ? c0 + u : nchunks - 1;
      v[u] = *reinterpret_cast<const f32x4*>(po + static_cast<size_t>(cidx) * (kBlk * kDim));
      mc[u] = ml[cidx * (2 * kBlk)];
      lc[u] = ml[cidx * (2 * kBlk) + kBlk];
    }
    float m_new = M;
#pragma unroll
    for (int u = 0; u < U; ++u) m_new = fmaxf(m_new, mc[u]);
    if (m_new == neg_inf()) continue;  // nothing but empty slices so far
    const float alpha = fast_exp2(M - m_new);
    M = m_new;
    L *= alpha;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float wgt = c0 + u < nchunks && mc[u] != neg_inf() ? fast_exp2(mc[u] - M) : 0.f;
      L += lc[u] * wgt;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += v[u][e] * wgt;
    }
  }
  const float inv = L > 0.f ? p.drop.rs / L : 0.f;  // (rs: 1, or the dropout scale)
  const size_t row = static_cast<size_t>(bh) * p.n + j * kBlk + q;
  if ((threadIdx.x & 15) == 0) p.LSE[row] = L > 0.f ? (M + fast_log2(L)) * kLn2 : neg_inf();
  if constexpr (BF16) {
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = static_cast<__bf16>(acc[e] * inv);
    *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.O) + row * kDim + d0) = v;
  } else {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = acc[e] * inv;
    *reinterpret_cast<f32x4*>(static_cast<float*>(p.O) + row * kDim + d0) = v;
  }
}

namespace {
// Reports a failed launch on stderr (the status code cannot carry the runtime's reason).
bool launch_failed(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return false;
  fprintf(stderr, "bigbird: launch of %s failed: %s\n", what, hipGetErrorString(e));
  return true;
}
}  // namespace

int launch_fwd(const FwdParams& p, bool bf16, hipStream_t stream) {
  if (bf16) {
    const int st = launch_fwd_bf16_main(p, stream);
    if (st != BB_OK) return st;
  } else if (rows_f32_fwd(p.BH, p.nb, p.g, p.w, p.r, p.kmask != nullptr, p.drop.thr != 0)) {
    hipLaunchKernelGGL(fwd_rows_f32, dim3(own_grid(p.BH, p.nb)), dim3(kRowsThreadsF32), 0, stream, p);
    return launch_failed("fwd_rows_f32") ? BB_ERR_LAUNCH : BB_OK;
  } else {
    const unsigned grid = DieItems(p.BH, p.split.items_per_bh).grid();
    if (grid == 0) return BB_OK;
    hipLaunchKernelGGL(fwd_kernel_f32, dim3(grid), dim3(kThreadsF32), 0, stream, p);
    if (launch_failed("fwd_kernel_f32")) return BB_ERR_LAUNCH;
  }
  const int rows_per_bh = p.cmb_g_rows + p.cmb_s_rows;
  if (rows_per_bh > 0) {
    const unsigned cgrid = static_cast<unsigned>(p.BH) * rows_per_bh * kCombineSplit;
    if (bf16)
      hipLaunchKernelGGL(fwd_combine_kernel<true>, dim3(cgrid), dim3(kCombineThreads), 0, stream, p);
    else
      hipLaunchKernelGGL(fwd_combine_kernel<false>, dim3(cgrid), dim3(kCombineThreads), 0, stream, p);
    if (launch_failed("fwd_combine_kernel")) return BB_ERR_LAUNCH;
  }
  return BB_OK;
}

}  // namespace bb
