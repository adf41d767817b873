// Launch interface of the forward kernels (internal to the library).
#ifndef BB_FWD_KERNELS_H_
#define BB_FWD_KERNELS_H_

#include "dropout.h"
#include "kernel_common.h"

namespace bb {

// Work decomposition of the bf16 forward.  Workgroups have four independent waves (eight in launches of medium size).
//   global workgroup: one global query block x up to 64 key blocks, 16 (8) per wave, merged in LDS;
//   persistent workgroup: its waves take the die's other items (non-global query block x slice
//   of up to 16 key blocks: 8 at the ITC base pattern) in turn, wave w the items w, w + W, ...
// A global row longer than 64 key blocks takes several workgroups whose merged partial
// results go through the merge kernel, as do sparse rows with more than one slice.
constexpr int kGlobalWaveLen = 16;  // most key blocks a wave of a global workgroup takes
// Items a wave may put on its list of items to redo before it stops taking others: a lane of one register
// each, less the two that can still be in flight (the item in work and the next).
constexpr int kListedItems = 62;
constexpr int kCounterStride = 32;  // ints between the item counters of two dies (a 128-byte line each)
struct Bf16Geom {
  int waves;     // of a workgroup: 4, or 8
  int by_row;    // small launches: every row is done the way global rows are, a workgroup per row; no
                 // persistent workgroups
  int sw_len;    // by_row: key blocks per wave of a non-global row
  int gw_len;    // key blocks per wave of a global workgroup: 16; 8 when the whole grid fits the chip at once (then
                 // the global rows alone would set the run time); an equal share of the row in small launches and for short rows
  int ng;        // workgroups per global row: ceil(nb / (waves * gw_len))
  int cs;        // slices per non-global row: ceil(min(g + w + r, nb) / 16)
  int n_sitems;  // (nb - g) * cs
  int p_wgs;     // persistent workgroups per die: their waves share out the die's non-global items
  int g_wgs;     // row workgroups per (batch, head): g * ng of global rows, then, by_row, the other rows
  int bh_rounds; // ceil(B*H / 8)
};

// The decomposition of a launch.  masked: there is a padding mask.
inline Bf16Geom make_bf16_geom(int BH, int nb, int g, int w, int r, bool masked) {
  Bf16Geom q;
  const int sparse_ub = longest_sparse_list(nb, g, w, r);
  auto cut = [](int n, int by) { return (n + by - 1) / by; };
  // a wave takes up to 16 key blocks of a non-global row; wider patterns are sliced
  q.cs = sparse_ub > kGlobalWaveLen ? cut(sparse_ub, kGlobalWaveLen) : 1;
  q.n_sitems = (nb - g) * q.cs;
  q.bh_rounds = cut(BH, kXcd);
  q.waves = 4;
  q.by_row = 0;
  q.sw_len = 0;
  // Global rows: 16 key blocks per wave (up to 64 per workgroup, merged in LDS).  When every workgroup of the launch is
  // resident at once (two per CU, 32 CUs per die) the longest one sets the run time: then 8 per wave, by several workgroups
  // to a row, whose partial results the merge kernel combines.
  constexpr int kHalfLen = kGlobalWaveLen / 2;
  const bool halves = nb > 4 * kHalfLen && q.bh_rounds * (g * cut(nb, 4 * kHalfLen) + cut(q.n_sitems, 4)) <= 64;
  q.gw_len = halves ? kHalfLen : kGlobalWaveLen;
  q.ng = cut(nb, 4 * q.gw_len);
  // With a workgroup for every row, up to 11 blocks per wave in one workgroup cost less than the merge launch (us, one workgroup
  // to a global row and two: 4 slices of n = 2560 11.9 and 13.8, dropout 22.8 and 22.6; n = 3200 14.4 and 14.1, 28.1 and 22.7).  Under a mask
  // the blocks that are left may all be the first wave's (4 of n = 3200, half of it padded, 21.1 and 14.5).  Where lists are long and
  // only one workgroup to a global row leaves room for one to every row, dealing them out wins (6 of n = 3072, lists of 16: 16.4 and
  // 21.9, dropout 29.1 and 39.6; 5 of n = 3200 with room for either 15.4 and 18.9, 28.5 and 28.8).
  auto all_rows = [&](int ng) { return static_cast<long long>(BH) * (g * ng + nb - g) <= 288 && sparse_ub <= 4 * kGlobalWaveLen; };
  const bool whole_rows = (!masked && nb <= (sparse_ub > 12 ? 52 : 44)) || (sparse_ub > 12 && nb <= 4 * kGlobalWaveLen && !all_rows(q.ng));
  const int row_ng = whole_rows ? 1 : q.ng;
  // Eight waves to a workgroup, where every workgroup is resident at once (a die has 32 CUs of eight waves) and the longest
  // wave sets the run time: a global row's list is then dealt out to eight waves, up to 64 blocks without a merge launch.  us of
  // four waves (16 blocks of a global row each; from 33 blocks on 8, several workgroups to a row and a merge launch) and what eight take
  // of that, plain / dropout, by the lists of the other rows (lists of 4, 8, 12 and 16 blocks):
  //   n = 1024 .. 2048, wgs(4) <= 32 (one wave to a SIMD)  16 / 34 us: 0.73 / 0.57, 1.03 / 0.91, 1.31 / 1.22, 1.45 / 1.44; 7 blocks 0.95 / 0.82
  //   n = 1024 .. 2048, past that                          18 .. 25 / 35 .. 50 us: 0.66 / 0.55, 0.84 / 0.76, 0.95 / 0.92, 1.05 / 1.05
  //     (just past it, 36 slices of n = 1280, wgs(4) = 33: 1.02 / 0.90 with 8 blocks, 1.24 / 1.15 with 11, 1.30 / 1.22 with 12)
  //   n = 2304 .. 4096, wgs(4) <= 32                       14 .. 21 / 23 .. 40 us: 0.88 .. 1.13 / 0.95 .. 1.3, 1.09 / 1.23, 1.17 / 1.29, 1.22 / 1.33
  //   n = 2304 .. 4096, past that                          15 .. 36 / 24 .. 59 us: 0.74 .. 0.97 / 0.79 .. 1.1, 0.83 / 0.9, 0.84 .. 0.97 / 0.92 .. 1.09,
  //     0.98 .. 1.02 / 1.2 up to wgs(4) = 48 and 0.85 .. 0.95 / 0.91 .. 1.15 from 54 on
  //   n > 4096 (a merge launch with either): 1.10 .. 1.16 / 1.25, 0.98 / 1.0, 0.96 .. 1.06 / 1.0 .. 1.15, and 1.0 .. 1.25 under a mask
  // Past wgs(8) = 32 the global rows wait for each other (64 slices of n = 1280, 34: 22.7 and 31.9 us).  Rows below 16 blocks are
  // dealt out in quarters to four waves, and eighths gain nothing (64 of n = 896 16.0 / 25.6 and 17.9 / 31.0 us, 48 of n = 960
  // 12.4 / 22.0 and 17.3 / 30.9).  Under a mask short lists come out shorter, and fill four waves less (7 blocks 0.7 .. 1.3).
  auto eight_waves = [&](int wgs4, int wgs8) {
    if (g == 0 || nb < kGlobalWaveLen || wgs8 > 32) return false;
    if (nb > 8 * kHalfLen) return !masked && sparse_ub >= 8 && sparse_ub <= 12 && wgs4 > 44;
    if (sparse_ub > 12) return nb > 4 * kHalfLen && wgs4 > 52;
    return wgs4 > (sparse_ub > 8 ? 33 : 32) || (nb <= 4 * kHalfLen && sparse_ub <= (masked ? 5 : 7));
  };
  // the workgroups a die gets with half as many blocks per wave, as they are launched: the items of its slices together
  auto wgs = [&](int waves) { return q.bh_rounds * g * cut(nb, waves * kHalfLen) + cut(q.bh_rounds * q.n_sitems, waves); };
  if (all_rows(row_ng)) {
    // Small launches, about a workgroup per CU: all rows that way, the key list of each dealt out to four
    // waves.  12 heads, n = 512 / 1024 / 1536: 12.2 -> 7.2, 12.4 -> 8.7, 12.5 -> 11.9 us; past that CUs have
    // two such workgroups and single waves with whole rows win (n = 2048, 384 rows: 12.7 against 17.5).
    q.by_row = 1;
    q.ng = row_ng;
  } else if (eight_waves(wgs(4), wgs(8))) {
    q.waves = 8;
    q.gw_len = kHalfLen;
    q.ng = cut(nb, 8 * kHalfLen);
  }
  q.g_wgs = g * q.ng;
  if (q.by_row) {
    q.sw_len = sparse_ub > q.waves ? cut(sparse_ub, q.waves) : 1;
    q.g_wgs += nb - g;
    q.cs = 1;
  }
  // A global row of one workgroup: an equal share for each wave in small launches and for short rows (96 slices of
  // n = 512 15.5 -> 14.1 us, 144 of n = 768 26.2 -> 25.1); longer ones keep 16 blocks per wave, which leaves
  // other waves a SIMD of their own meanwhile (96 of n = 1024 27.0 against 27.6 in quarters, 72 of n = 1536 26.6
  // against 26.9, 36 of n = 3072 26.9 against 27.2).
  if (q.ng == 1 && (q.by_row || q.waves == 8 || nb < kGlobalWaveLen)) q.gw_len = cut(nb, q.waves);
  {
    // Persistent workgroups: as many as stay resident beside the global-row workgroups (a die
    // holds 256 waves of this kernel: eight per CU), at most one wave per item.
    const int slots_per_die = 256 / q.waves;
    const int n_global = q.bh_rounds * q.g_wgs;
    const int want = cut(q.bh_rounds * q.n_sitems, q.waves);
    int avail = slots_per_die - n_global;
    if (avail < slots_per_die / 4) avail = slots_per_die / 2;  // the global rows alone fill the die: queue behind them
    q.p_wgs = want < avail ? want : avail;
    // a wave lists the items it has to redo by the exact recurrence in one register: no wave may be
    // given more than the list takes, and together the lists have to take every item, whatever that
    // does to residency
    const int floor_wgs = cut(q.bh_rounds * q.n_sitems, q.waves * kListedItems);
    if (q.p_wgs < floor_wgs) q.p_wgs = floor_wgs;
  }
  return q;
}

struct FwdParams {
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  float* LSE;
  const int32_t* rand_idx;
  const uint8_t* kmask;
  float* part_o;   // [slots][64][64] un-normalised partial outputs of split rows
  float* part_ml;  // [slots][2][64]  their running maxima (log2 units) and sums
  int B, H, BH, n, nb, g, w, r, global_mode;
  float c;  // scale * log2(e)
  RowSplit split;  // decomposition used by the fp32 kernel
  Bf16Geom geo;    // decomposition used by the bf16 kernel
  // rows whose slices the merge kernel combines: cmb_g_rows global rows of cmb_g_n slices each
  // (slots first), then cmb_s_rows non-global rows of cmb_s_n slices; slots_per_bh in total
  int cmb_g_rows, cmb_g_n, cmb_s_rows, cmb_s_n, slots_per_bh;
  Dropout drop;  // attention dropout (thr == 0: none)
  int skip_q;    // query blocks without a valid position (in kmask) are not computed: O = 0, LSE = -inf
  int dyn;       // bf16 kernel: waves claim their items after the first from the die's counter
  int* counters; // [8 * kCounterStride] one per die, zeroed by a small launch before the kernel (dyn != 0 only)
};

// Enqueues the fused forward kernel and, if any row is split, the merge kernel.
int launch_fwd(const FwdParams& p, bool bf16, hipStream_t stream);

// The tuned bf16 main kernel (defined in fwd_bf16.hip); launch_fwd calls it.
int launch_fwd_bf16_main(const FwdParams& p, hipStream_t stream);

}  // namespace bb
#endif  // BB_FWD_KERNELS_H_
