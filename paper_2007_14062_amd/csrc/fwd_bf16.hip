// bf16 forward kernel: the tuned path of the BERT-shaped workloads.
//
// Same mathematics as the fp32 kernel (eq. (AT) per head on the App. D pattern),
// organised around what limits it on this chip at d = 64: the vector port (one
// exponential per score) and the matrix pipe are within a few percent of each other,
// so every vector instruction per score counts.
//   * One wavefront owns one work item at a time: a 64-query block against a slice of
//     its key blocks (up to 16).  Waves never wait for each other inside the key-block
//     loop.  Per die, the first workgroups take one global query block each (key list
//     dealt out 16 blocks per wave, the four waves' results merged in LDS: no partial
//     results in HBM and no second kernel for up to 64 key blocks; longer rows take
//     several workgroups plus the merge kernel; launches of medium size, where it pays
//     (make_bf16_geom): 8 blocks per wave and workgroups of eight waves, which took 24 slices of
//     n = 4096 from 24.0 us, a merge launch in them, to 19.7).  The other workgroups stay for the whole
//     launch: their waves share out the die's non-global items round robin and run them
//     as one uninterrupted stream of block pairs -- the next item's query tile and first
//     K tile ride at the end of this item's K and V tile streams, so the matrix pipe
//     only idles for the item's output.
//   * Softmax without a running maximum.  A probability is 2^(score * scale*log2(e)): one
//     multiplication and one v_exp_f32 per score, no row maximum, no accumulator rescale.
//     Softmax is shift invariant and fp32/bf16 carry eight exponent bits, so a fixed
//     reference of 0 is exact as long as the row sum stays inside [2^-40, 2^60]; a wave
//     checks that at the end of its item and, if a row left the range (logits beyond about
//     +-28 in natural units), puts the item on a list that it works off afterwards with the
//     classical running-maximum recurrence (running_item).  Both paths give the same un-normalised (reference, sum,
//     O~) triple to the common epilogue.  (Folding the factor into the query operand would
//     save the multiplication, but the operand would have to be rounded to bf16 again: that
//     perturbs a logit by up to 2^-8 of its size, four times the error of everything else in
//     LSE, and the backward pass, which recomputes the logits exactly, then sees rows whose
//     probabilities do not sum to one -- measured: gradient errors three times as large.)
//   * Row sums come from the matrix pipe as well: one small MFMA per 16 keys multiplies
//     the probabilities (already in operand layout) by a matrix of ones and zeros
//     (RowSumOperand).  That takes sixteen additions per unit off the vector port.
//   * The block pair is cut into four units (32 keys x 32 queries each) that flow through
//     a three-stage software pipeline inside the wave: scores of unit u+1 on the matrix
//     pipe, exponentials of unit u on the vector ALU, P V of unit u-1 on the matrix pipe
//     again.  The pipeline runs across key-block and item boundaries with one
//     straight-line body (pair_step) whose issue order (one MFMA, two exponentials, a
//     conversion, ...) is pinned with scheduling group barriers.  Every K and V^T operand
//     fetched from LDS feeds two MFMAs (two query tiles), which halves the LDS traffic
//     per flop.
//   * K and V tiles go global -> LDS directly (no registers in between), one 8 KB
//     buffer each, handled as 32-key halves: as soon as a half has been read out into
//     operand registers the same half of the next key block is requested, so a load has
//     three quarters of a block pair to land.
//   * V^T operands come from the transposing LDS read; the LDS layout is swizzled so
//     that neither read pattern has bank conflicts.
//   * Items with a block that has padded keys inside take the recurrence, in the same streams and with a pipelined
//     body of its own (running_pair): its row sums are fp32 sums of the probabilities before their rounding, and
//     the largest probability of a row is 1 and not rounded.  (Against the fixed reference LSE is off by up
//     to 2^-8 where one key holds a row, and O by 2.33e-3 -- 2-norm, normal inputs, rows of 454 keys -- where the
//     recurrence has 2.18e-3.  A maximum of the whole row found in a pass of its own gives 2.23e-3: the maxima on
//     the way there are exact too.)  What bounds it is the vector port, 410 instructions a pair (98 more where keys
//     are padded) and the body without a maximum 206, matrix instructions included: 230 leading global tokens, where
//     every item has such a block, 74.6 -> 55.1 us (42 with 256); 8 sequences of 1024 .. 4096 valid positions, 12 heads, n =
//     4096, 85.8 -> 73.9 us, and with padded query blocks skipped 89.0 -> 58.8.  (The recurrence had been one pair
//     after another and its items a list worked off at the end, while other waves had nothing left to do.)  The order of issue inside its slots, pinned in
//     six ways, made no difference beyond 1 us and is left to the compiler.
//     The list builder leaves the validity bits of such blocks in LDS, so that no pair waits for the mask.
//   * The two waves of a SIMD get their issue priority from the pairs they still have to
//     do, so that they finish together (set_issue_priority).
//   * Instances of the kernel: without a padding mask (everything above and nothing else); with
//     one; kOptions, launched when a call asks for fully padded query blocks to be skipped
//     (BB_SKIP_PADDED_QUERY_BLOCKS: their rows are written as zeros and the waves claim the
//     other items from a counter per die, global-row waves included once their row is done); and
//     kDrop for attention dropout, with or without these.  There every item takes the recurrence,
//     and the keep mask of dropout.h is applied to the converted pairs that multiply V.
//     (A pipelined body with the mask inside measured 46 against 53 us at 48 slices of n = 3072, padded
//     blocks skipped; against a fixed reference the largest probability of a row is rounded: O is off by
//     2.33e-3 where the recurrence has 2.19e-3, and the slices of a cut row need two sums each.)
// -DBB_STAMPS builds a development variant that writes per-wave time stamps into the
// partial-result workspace (which must then hold 128 bytes per wave of the launch); the
// library proper is built without it.
#include "fwd_epilogue.h"
#include "key_list.h"
#include "tile_ops.h"

#include <cstdio>

namespace bb {

namespace {

// Instances of the kernel: no padding mask; a padding mask; a padding mask and skipped query blocks;
// attention dropout with any of these.
enum { kPlain = 0, kMasked = 1, kOptions = 2, kDrop = 3 };

// Row sums of the reference-free path must stay inside [kSumLo, kSumHi] (see the file header).
constexpr float kSumLo = 0x1p-40f;
constexpr float kSumHi = 0x1p60f;

__device__ __forceinline__ void zero_acc(f32x16 (&a)[2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[t][r] = 0.f;
}


// Issue priority of the wave by the block pairs it still has to do, in steps of four pairs: the
// two waves of a SIMD would otherwise be served oldest first, the older one would finish pairs
// ahead of the younger, and the younger would do its last pairs alone at a little more than half
// the throughput the SIMD has with two waves.  (Priority is an immediate operand.)
__device__ __forceinline__ void set_issue_priority(int remaining_pairs) {
  const int pr = remaining_pairs >> 2;
  if (pr >= 3) {
    __builtin_amdgcn_s_setprio(3);
  } else if (pr == 2) {
    __builtin_amdgcn_s_setprio(2);
  } else if (pr == 1) {
    __builtin_amdgcn_s_setprio(1);
  } else {
    __builtin_amdgcn_s_setprio(0);
  }
}

// ---------------------------------------------------------------------------------------------
// The pipelined pair step.
//
// A block pair (64 queries x 64 keys) is four units u = (t, q): keys 32t .. 32t+31 against the
// query tile q (A: queries 0..31, B: 32..63), taken in the order (0,A) (0,B) (1,A) (1,B).
// Stage S(u): 4 MFMAs, S^T = K_t Q_q^T (keys along MFMA rows, a lane owns one query column).
// Stage E(u): 16 exponentials, 8 conversions to bf16 pairs.
// Stage P(u): 4 MFMAs, O_q^T += V_t^T P^T, the converted scores being the B operand as they are,
//             and 2 small MFMAs for the row sums.
// Slot k of the stream issues S(k+1), E(k), P(k-1).  Unit (0,A) of the next pair is therefore
// started in the last slot of this one, and P of unit (1,B) is finished in the first slot of
// the next pair (`sA`, `p3` carry them across).
//
// Operand registers: ka[t] (K half t, "straight" fragments), va[t] (V half t, transposed
// fragments).  Each is refilled from LDS in the slot after its last use, from the half tile that
// was requested three slots earlier; the request for the half after that follows as soon as the
// read has returned.  Tile loads outstanding at the start of a pair, oldest first:
// K(i+1).t0 and V(i).t1 (8 instructions).
// Blocks with padded keys inside never come here: such items take the recurrence (running_pair).
struct PairCtx {
  const char* lds_k;   // this wave's K and V tile buffers
  const char* lds_v;
  unsigned lds_k_a, lds_v_a;  // the same as LDS byte addresses (scalar)
  unsigned voff[2];
  int hf;
  float c;  // scale * log2(e)
};

__device__ __forceinline__ void unit_scores(const bf16x8 (&k)[4], const bf16x8 (&q)[4], f32x16& s) {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k[0], q[0], z, 0, 0, 0);
#pragma unroll
  for (int ks = 1; ks < 4; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k[ks], q[ks], s, 0, 0, 0);
}

// Row sums on the matrix pipe.  A B operand of the 32x32x16 product (lane: query lane % 32, eight
// keys chosen by lane / 32) is read by the 16x16x32 product as column lane % 16, key group
// lane / 16: groups 0 and 2 of column c are the two key halves of query c, groups 1 and 3 those of
// query c + 16.  With an A operand whose row m is one on the groups g with m + g even and zero on
// the others, even output rows hold the sums of queries 0..15 and odd rows those of queries
// 16..31, and the output layout (lane: column lane % 16, rows 4 (lane / 16) .. + 3) gives every lane
// the total of its own query: element 0 for lane % 32 < 16, element 1 otherwise.  The sums are
// those of the rounded probabilities, the same numbers that multiply V.
struct RowSumOperand {
  bf16x8 a;
  __device__ __forceinline__ explicit RowSumOperand(int lane) {
    const __bf16 v = static_cast<__bf16>((((lane & 15) + (lane >> 4)) & 1) ? 0.f : 1.f);
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = v;
  }
};
__device__ __forceinline__ float row_total(const f32x4& ls, int col) { return col < 16 ? ls[0] : ls[1]; }

// O^T += V_t^T P^T for one unit.
__device__ __forceinline__ void unit_pv(const bf16x8 (&v)[2][2], const bf16x8 (&pb)[2], f32x16 (&o)[2]) {
#pragma unroll
  for (int sgl = 0; sgl < 2; ++sgl)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
      o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt][sgl], pb[sgl], o[dt], 0, 0, 0);
}

// The same, and the unit's share of the row sums.
__device__ __forceinline__ void unit_pv(const bf16x8 (&v)[2][2], const bf16x8 (&pb)[2], f32x16 (&o)[2],
                                        const RowSumOperand& ones, f32x4& ls) {
#pragma unroll
  for (int sgl = 0; sgl < 2; ++sgl) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
      o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt][sgl], pb[sgl], o[dt], 0, 0, 0);
    ls = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.a, pb[sgl], ls, 0, 0, 0);
  }
}

// Probabilities of one unit as two B operands (16 keys each).  (The row sums are taken from these
// operands by unit_pv: sixteen additions per unit here, or eight packed bf16 dots -- which stall
// against the MFMAs in flight, measured 16 cycles each -- would sit on the vector port, which is
// the busier of the two pipes.)
__device__ __forceinline__ void unit_probs(const f32x16& s, float c, bf16x8 (&pb)[2]) {
#pragma unroll
  for (int sgl = 0; sgl < 2; ++sgl)
#pragma unroll
    for (int kk = 0; kk < 8; kk += 2) {
      const int r = sgl * 8 + kk;
      const float p0 = fast_exp2(s[r] * c);
      const float p1 = fast_exp2(s[r + 1] * c);
      const bf16x2 pk = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
      pb[sgl][kk] = pk[0];
      pb[sgl][kk + 1] = pk[1];
    }
}

// issue order of one slot: eight times (one MFMA, [LDS reads,] two exponentials), the two small
// row-sum MFMAs after the fourth and the eighth; the multiplications, conversions and lane reads
// fall where the scheduler puts them between those (pinning them too measured 1.5 % slower);
// nothing moves across the end of a slot
template <int DS_READS>
__device__ __forceinline__ void pin_slot() {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (u * 2 < DS_READS) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);  // two exponentials
    if (u == 3 || u == 7) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// One block pair.  The arithmetic and the memory requests are the same for every pair, so that
// one straight-line body serves them all: the first pair of an item finishes a predecessor that
// does not exist (p3 = 0 on entry, V fragments zeroed), the last one starts a successor that does
// not exist (scores of whatever the K fragments hold, never used) -- eight idle MFMAs per item
// instead of differently scheduled copies of the body -- and a stream that has run out of tiles
// delivers a tile nobody uses (see TileStreams).
// k1 / v1: global address of the tile that follows this pair's in the K / V stream; k2: the one
// after that in the K stream.
__device__ __forceinline__ void pair_step(const PairCtx& cx, const StraightOffsets& so, const TransposedOffsets& to,
                                          const bf16x8 (&qb)[2][4], bf16x8 (&ka)[2][4], bf16x8 (&va)[2][2][2],
                                          f32x16& sA, bf16x8 (&p3)[2], f32x16 (&o)[2][2],
                                          const RowSumOperand& ones, f32x4 (&ls)[2],
                                          const char* k1, const char* v1, const char* k2) {
  f32x16 sB, sC, sD;
  bf16x8 p0[2], p1[2], p2[2];

  // ---- slot 0: the reads issued in the previous slot (K.t1, V.t0 of this pair) have returned
  wait_lds_reads();
  half_load_async(k1, cx.lds_k_a, 1, cx.voff);
  half_load_async(v1, cx.lds_v_a, 0, cx.voff);
  unit_scores(ka[0], qb[1], sB);
  unit_pv(va[1], p3, o[1], ones, ls[1]);
  unit_probs(sA, cx.c, p0);
  pin_slot<0>();

  // ---- slot 1: K(i+1).t0 and V(i).t1 have landed
  wait_tile_loads<8>();
  read_straight_half(so, cx.lds_k, 0, ka[0]);
  read_transposed_half(to, cx.lds_v, 1, va[1]);
  unit_scores(ka[1], qb[0], sC);
  unit_pv(va[0], p0, o[0], ones, ls[0]);
  unit_probs(sB, cx.c, p1);
  pin_slot<12>();

  // ---- slot 2
  wait_lds_reads();
  half_load_async(k2, cx.lds_k_a, 0, cx.voff);
  half_load_async(v1, cx.lds_v_a, 1, cx.voff);
  unit_scores(ka[1], qb[1], sD);
  unit_pv(va[0], p1, o[1], ones, ls[1]);
  unit_probs(sC, cx.c, p2);
  pin_slot<0>();

  // ---- slot 3: K(i+1).t1 and V(i+1).t0 have landed
  wait_tile_loads<8>();
  read_straight_half(so, cx.lds_k, 1, ka[1]);
  read_transposed_half(to, cx.lds_v, 0, va[0]);
  unit_scores(ka[0], qb[0], sA);
  unit_pv(va[1], p2, o[0], ones, ls[0]);
  unit_probs(sD, cx.c, p3);
  pin_slot<12>();
}

// The same pair with the classical softmax recurrence: every probability is taken against the running maximum
// of its row, the sums are fp32 sums of the probabilities before their rounding.  For items with a block
// that has padded keys inside, for attention dropout, and for items whose row sums left the safe range of the
// reference-free path.
//
// The maximum of a row over the 64 keys of the pair has to be known before the first exponential, so the
// units go (0,A) (1,A) (0,B) (1,B) and the scores run two units ahead: slot k of the stream issues S(k+2), E(k), P(k-1).
// Entering a pair, s0 and s1 are the scores of (0,A) and (1,A), ka its K fragments, and outstanding are V(i) and
// K(i+1) (V(i).t0 oldest).
// Operand reads from two registers instead of the eight of StraightOffsets and TransposedOffsets: the others differ
// from them in single bits of the address (see tile_off_bf16), and three scores in flight leave no registers.
struct LeanOffsets {
  int s0, t0;
  __device__ __forceinline__ explicit LeanOffsets(int lane) : s0(StraightOffsets(lane).off[0]), t0(TransposedOffsets(lane).off[0][0]) {}
  __device__ __forceinline__ void straight_half(const char* tile, int t, bf16x8 (&f)[4]) const {
    const int base = lane_again(s0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) f[ks] = *reinterpret_cast<const bf16x8*>(tile + (base ^ (ks << 5)) + t * kHalfTile);
  }
  __device__ __forceinline__ void transposed_half(const char* tile, int t, bf16x8 (&f)[2][2]) const {
    const int base = lane_again(t0);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int sgl = 0; sgl < 2; ++sgl) {
        union { s16x4 half[2]; bf16x8 v; } u;
#pragma unroll
        for (int half = 0; half < 2; ++half)
          u.half[half] = lds_read_tr16(tile + (base ^ (dt << 6) ^ (half << 5)) + half * 1024 + (2 * t + sgl) * 2048);
        f[dt][sgl] = u.v;
      }
  }
};

struct RowState {
  float m[2], l[2];  // per query tile: reference exponent (base 2; the lane halves agree), this lane's share of the row sum
};

// Padded keys of a half block never count: selected, not added to (their scores may be anything).
__device__ __forceinline__ void drop_padded_scores(uint32_t bits, int hf, f32x16& s) {
  const uint32_t mine = bits >> (hf * 4);
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = ((mine >> acc_row(r, 0)) & 1) ? s[r] : neg_inf();
}

// Running maximum of the rows of a query tile over another 64 keys; what is summed so far is rescaled to it.
__device__ __forceinline__ float raise_reference(const f32x16& s0, const f32x16& s1, float c, float& m, float& l,
                                                 f32x16 (&o)[2]) {
  // (the maximum that keeps a NaN: one instruction for three values, where fmaxf first quiets the scores; a row with a
  // NaN among its scores has a NaN among its probabilities either way)
  float x[2] = {s0[0], s1[0]};
#pragma unroll
  for (int r = 1; r < 15; r += 2) {
    x[0] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x[0], s0[r]), s0[r + 1]);
    x[1] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x[1], s1[r]), s1[r + 1]);
  }
  x[0] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x[0], s0[15]), s1[15]);
  const float mloc = half_max(__builtin_elementwise_maximum(x[0], x[1])) * c;
  const float m_new = fmaxf(m, mloc);
  const float m_use = m_new == neg_inf() ? 0.f : m_new;
  const float alpha = fast_exp2(m - m_use);  // 0 while m is still -inf
  m = m_new;
  l *= alpha;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
  return m_use;
}

// What attention dropout needs of an item: drop_first of the keys of this lane's two rows of the keep mask.
struct DropRows {
  uint32_t rk[2];
  uint32_t thr;
};

// Probabilities of one unit against a reference, as two B operands; their sum before rounding goes to l.
// drop_words: the unit's key words (drop_unit_words).
template <bool kDropout>
__device__ __forceinline__ void unit_probs_against(const f32x16& s, float c, float m_use, float& l, bf16x8 (&pb)[2],
                                                   uint32_t drop_rk, uint32_t drop_thr, const uint32_t* drop_words) {
  float sum[2] = {0.f, 0.f};
#pragma unroll
  for (int sgl = 0; sgl < 2; ++sgl) {
#pragma unroll
    for (int kk = 0; kk < 8; kk += 2) {
      const int r = sgl * 8 + kk;
      const float p0 = fast_exp2(__builtin_fmaf(s[r], c, -m_use));
      const float p1 = fast_exp2(__builtin_fmaf(s[r + 1], c, -m_use));
      sum[0] += p0;  // (the row sums are those of the undropped probabilities)
      sum[1] += p1;
      bf16x2 pk = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
      if constexpr (kDropout)
        pk = __builtin_bit_cast(bf16x2, drop_apply(__builtin_bit_cast(uint32_t, pk), drop_keep_pair(drop_doubled(drop_rk ^ drop_words[r >> 1]), drop_thr)));
      pb[sgl][kk] = pk[0];
      pb[sgl][kk + 1] = pk[1];
    }
  }
  l += sum[0] + sum[1];
}

// key_bits: validity bits of the pair's keys if `cut`, else not read.  kblock: its key block (dropout only).
// kLast: nothing follows, so nothing is requested and no scores run ahead; k_ahead: the pair before it has requested a K tile.
template <bool kMask, bool kDropout, bool kLast = false>
__device__ __forceinline__ void running_pair(const PairCtx& cx, const LeanOffsets& lo,
                                             const bf16x8 (&qb)[2][4], bf16x8 (&ka)[2][4], bf16x8 (&va)[2][2][2],
                                             f32x16& s0, f32x16& s1, bf16x8 (&p3)[2], f32x16 (&o)[2][2], RowState& rs,
                                             const DropRows& drop, uint32_t* drop_table, uint32_t kblock, bool cut, const uint32_t* key_bits,
                                             const char* k2, const char* v1, bool k_ahead = true) {
  f32x16 sB0, sB1;
  bf16x8 p0[2], p1[2], p2[2];
  uint32_t vb[2] = {~0u, ~0u};
  if constexpr (kDropout) drop_key_words(drop_table, kblock, lane_again(lane_id()));
  if (kMask && cut) {
    vb[0] = key_bits[0];
    vb[1] = key_bits[1];
    drop_padded_scores(vb[0], cx.hf, s0);
    drop_padded_scores(vb[1], cx.hf, s1);
  }
  // ---- slot 0: (0,A).  V.t0 has landed; K.t1 of this pair (read in the previous pair) is in registers
  wait_lds_reads();
  if (k_ahead)
    wait_tile_loads<12>();
  else
    wait_tile_loads<4>();
  unit_pv(va[1], p3, o[1]);
  unit_scores(ka[0], qb[1], sB0);
  float mu = raise_reference(s0, s1, cx.c, rs.m[0], rs.l[0], o[0]);
  lo.transposed_half(cx.lds_v, 0, va[0]);
  unit_probs_against<kDropout>(s0, cx.c, mu, rs.l[0], p0, drop.rk[0], drop.thr, drop_unit_words(drop_table, 0, cx.hf));
  __builtin_amdgcn_sched_barrier(0);

  // ---- slot 1: (1,A).  V.t1 and K(i+1).t0 have landed
  wait_lds_reads();
  if constexpr (!kLast) {
    half_load_async(v1, cx.lds_v_a, 0, cx.voff);
    wait_tile_loads<8>();
  } else if (k_ahead) {
    wait_tile_loads<4>();  // (out are K.t0, V.t1, K.t1)
  } else {
    wait_tile_loads<0>();
  }
  unit_scores(ka[1], qb[1], sB1);
  unit_pv(va[0], p0, o[0]);
  if constexpr (!kLast) lo.straight_half(cx.lds_k, 0, ka[0]);
  lo.transposed_half(cx.lds_v, 1, va[1]);
  unit_probs_against<kDropout>(s1, cx.c, mu, rs.l[0], p1, drop.rk[0], drop.thr, drop_unit_words(drop_table, 1, cx.hf));
  asm volatile("" : "+v"(p1[0]), "+v"(p1[1]), "+v"(rs.l[0]));  // (made here, not behind the branch)
  __builtin_amdgcn_sched_barrier(0);

  // ---- slot 2: (0,B).  K(i+1).t1 has landed
  if (kMask && cut) {
    drop_padded_scores(vb[0], cx.hf, sB0);
    drop_padded_scores(vb[1], cx.hf, sB1);
  }
  wait_lds_reads();
  if constexpr (!kLast) {
    half_load_async(k2, cx.lds_k_a, 0, cx.voff);
    half_load_async(v1, cx.lds_v_a, 1, cx.voff);
    wait_tile_loads<12>();
  }
  unit_pv(va[1], p1, o[0]);
  if constexpr (!kLast) unit_scores(ka[0], qb[0], s0);
  mu = raise_reference(sB0, sB1, cx.c, rs.m[1], rs.l[1], o[1]);
  if constexpr (!kLast) lo.straight_half(cx.lds_k, 1, ka[1]);
  unit_probs_against<kDropout>(sB0, cx.c, mu, rs.l[1], p2, drop.rk[1], drop.thr, drop_unit_words(drop_table, 0, cx.hf));
  __builtin_amdgcn_sched_barrier(0);

  // ---- slot 3: (1,B)
  wait_lds_reads();
  if constexpr (!kLast) {
    half_load_async(k2, cx.lds_k_a, 1, cx.voff);
    unit_scores(ka[1], qb[0], s1);
  }
  unit_pv(va[0], p2, o[1]);
  unit_probs_against<kDropout>(sB1, cx.c, mu, rs.l[1], p3, drop.rk[1], drop.thr, drop_unit_words(drop_table, 1, cx.hf));
  asm volatile("" : "+v"(p3[0]), "+v"(p3[1]), "+v"(rs.l[1]));
  __builtin_amdgcn_sched_barrier(0);
}

// LDS of a workgroup of W waves (the cold paths below are separate functions; an instance holds the arrays it names).
template <int W>
__device__ __forceinline__ auto tiles_of(int wv) -> char (&)[2 * kTile] {  // per wave: K tile, V tile
  __shared__ __attribute__((aligned(1024))) char tiles[W][2 * kTile];
  return tiles[wv];
}
template <int W>
__device__ __forceinline__ int* klist_of(int wv) {
  __shared__ int klist[W][kGlobalWaveLen];
  return klist[wv];
}
// validity bits of the keys of listed blocks that have padded keys inside, of the item in work and of the next one
template <int W>
__device__ __forceinline__ auto key_bits_of(int wv, int set) -> uint32_t (&)[kGlobalWaveLen][2] {
  __shared__ uint32_t key_bits[W][2][kGlobalWaveLen][2];
  return key_bits[wv][set];
}
// dropout: key words of the pair in work
template <int kMode, int W>
__device__ __forceinline__ uint32_t* drop_words_of(int wv) {
  if constexpr (kMode == kDrop) {
    __shared__ __attribute__((aligned(16))) uint32_t words[W][32];
    return words[wv];
  }
  return nullptr;
}
// rows by a workgroup: does a wave's share hold a cut block?
template <int W>
__device__ __forceinline__ int* row_cut() {
  __shared__ int cut[W];
  return cut;
}
// their per-wave exponents and sums
template <int W>
__device__ __forceinline__ float* merge_m(int wv) {
  __shared__ float m[W][kBlk];
  return m[wv];
}
template <int W>
__device__ __forceinline__ float* merge_l(int wv) {
  __shared__ float l[W][kBlk];
  return l[wv];
}

// What a wave knows about itself and its LDS.
template <int W>
struct WaveCtx {
  int lane, wv, hf, col;
  char* lds_kv;  // this wave's 16 KB: K buffer, then V buffer
  char* lds_k;
  char* lds_v;
  int* klist;
  PairCtx cx;
  __device__ __forceinline__ explicit WaveCtx(float c, int lane_ = lane_id()) {
    lane = lane_;
    wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform, and the compiler should know
    hf = lane >> 5;
    col = lane & 31;
    lds_kv = tiles_of<W>(wv);
    lds_k = lds_kv;
    lds_v = lds_kv + kTile;
    klist = klist_of<W>(wv);
    cx.lds_k = lds_k;
    cx.lds_v = lds_v;
    cx.hf = hf;
    cx.c = c;
    half_load_offsets(lane, cx.voff);
    cx.lds_k_a = __builtin_amdgcn_readfirstlane(lds_addr(lds_k));
    cx.lds_v_a = __builtin_amdgcn_readfirstlane(lds_addr(lds_v));
  }
};

// Workgroup id -> work.  id % 8 is the die (XCD) the hardware dispatches to; each die gets
// whole (batch, head) slices so that a slice's K and V stay in its L2.  The first workgroups
// of a die take one global query block each (the longest items: 16 key blocks per wave).
// The others stay for the whole launch: wave w of the die's persistent waves takes the
// non-global items w, w + wave_stride, ... of the die, in (slice, query block) order, so that
// all waves start at once and nearly all end together.
template <int W>
struct Sched {
  int xcd;
  unsigned wg;        // workgroup number inside the die
  unsigned n_gpart;   // global-row workgroups of the die
  bool by_row;        // a constant of the kernel
  bool global_wg;     // a row by the whole workgroup (global rows; by_row: every row)
  int row_bh, row_idx;  // which one
  bool row_ok;
  int n_items_die;    // non-global items of the die
  int wave_stride;    // persistent waves of the die
  __device__ __forceinline__ explicit Sched(const FwdParams& p, bool by_row) {
    xcd = blockIdx.x % kXcd;
    wg = blockIdx.x / kXcd;
    n_gpart = static_cast<unsigned>(p.geo.bh_rounds) * p.geo.g_wgs;
    this->by_row = by_row;
    if (by_row) {
      global_wg = true;
      row_ok = DieItems(p.BH, p.geo.g_wgs).decode(blockIdx.x, &row_bh, &row_idx);
    } else {
      global_wg = wg < n_gpart;
      if (global_wg) {  // (two divisions that the other waves' first loads need not wait for)
        row_bh = static_cast<int>(wg / p.geo.g_wgs * kXcd + xcd);
        row_idx = static_cast<int>(wg % p.geo.g_wgs);
        row_ok = row_bh < p.BH;
      }
    }
    const int n_bh_die = xcd < p.BH ? (p.BH - xcd + kXcd - 1) / kXcd : 0;
    n_items_die = n_bh_die * p.geo.n_sitems;
    wave_stride = p.geo.p_wgs * W;
  }
};

// One work item as the kernel sees it between its phases.
struct Item {
  int bh, j;           // (batch, head) slice and query block
  int chunk, nchunks;  // slice of the row's key-block list, and how many there are
  int slot;            // partial-result slot (nchunks > 1)
  int cnt;             // key blocks in this slice
  int kl;              // the list: lane t holds entry t % 16
  unsigned partial;    // bit t: entry t has padded keys inside; its validity bits are in the wave's key_bits.  Not 0: takes the
                       // running maximum (running_pair)
  int bits;            // which of the wave's two sets of key_bits is its
  bool skipped;        // query block without a valid position, not to be computed (cnt = 0)
};

// Global addresses of an item's tiles (wave uniform, scalar arithmetic).
struct ItemTiles {
  const char* kbase;
  const char* vbase;
  const char* qtile;
  int kl;
  __device__ __forceinline__ ItemTiles(const FwdParams& p, const Item& it) {
    const size_t bh_row0 = static_cast<size_t>(it.bh) * p.n;
    kbase = static_cast<const char*>(p.K) + bh_row0 * (kDim * 2);
    vbase = static_cast<const char*>(p.V) + bh_row0 * (kDim * 2);
    qtile = static_cast<const char*>(p.Q) + (bh_row0 + it.j * kBlk) * (kDim * 2);
    kl = it.kl;
  }
  __device__ __forceinline__ const char* ktile(int i) const {
    return kbase + static_cast<size_t>(__builtin_amdgcn_readlane(kl, i)) * kTile;
  }
  __device__ __forceinline__ const char* vtile(int i) const {
    return vbase + static_cast<size_t>(__builtin_amdgcn_readlane(kl, i)) * kTile;
  }
};

// Item number -> item with its key-block list (for a global-row workgroup: the wave's share of
// the row).  All loads here are waited for before the function returns (scalar loads inside
// their asm statement, the others by the compiler), so tile loads in flight are at most delayed.
// Its first part: which row, which slice of the row's list (arithmetic only, no memory access).
template <int W>
__device__ __forceinline__ void item_coords(const FwdParams& p, const WaveCtx<W>& w, const Sched<W>& sc, int t, Item& it,
                                            int& list_lo, int& list_len, bool& row_global) {
  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  const Bf16Geom& geo = p.geo;
  if (sc.global_wg) {
    it.bh = sc.row_bh;
    const int n_glob = pat.g * geo.ng;
    if (sc.by_row && sc.row_idx >= n_glob) {
      row_global = false;
      it.j = pat.sparse_block(sc.row_idx - n_glob);
      it.chunk = 0;
      it.nchunks = 1;
      it.slot = 0;
      list_lo = w.wv * geo.sw_len;
      list_len = geo.sw_len;
      return;
    }
    const int row = sc.row_idx / geo.ng, u = sc.row_idx % geo.ng;
    row_global = true;
    it.j = pat.global_block(row);
    it.chunk = u;
    it.nchunks = geo.ng;
    it.slot = it.bh * p.slots_per_bh + row * geo.ng + u;
    list_lo = (u * W + w.wv) * geo.gw_len;
    list_len = geo.gw_len;
  } else {
    // (item order inside a die: slice by slice, so that a slice's K and V stay in the L2 while its
    // rows run -- also when items are claimed: row by row across the slices, which would put the
    // rows that are not computed last, measured 52.8 against 49.2 us at the key-padding workload)
    it.bh = (t / geo.n_sitems) * kXcd + sc.xcd;
    const int sitem = t % geo.n_sitems;
    row_global = false;
    it.j = pat.sparse_block(sitem / geo.cs);
    it.chunk = sitem % geo.cs;
    it.nchunks = geo.cs;
    it.slot = it.bh * p.slots_per_bh + p.cmb_g_rows * p.cmb_g_n + sitem;
    list_lo = it.chunk * kGlobalWaveLen;  // up to 16 key blocks per item (8 at the ITC base pattern)
    list_len = kGlobalWaveLen;
  }
}

__device__ __forceinline__ const char* query_tile(const FwdParams& p, int bh, int j) {
  return static_cast<const char*>(p.Q) + (static_cast<size_t>(bh) * p.n + static_cast<size_t>(j) * kBlk) * (kDim * 2);
}

// kMode (here and below): the instance of the kernel.  kPlain knows no padding mask, kMasked does,
// kOptions also skipped query blocks, kDrop attention dropout with or without these.  An instance holds no code of the
// others, so its registers and schedule are its own.
template <int kMode, int W>
__device__ __forceinline__ void make_item(const FwdParams& p, const WaveCtx<W>& w, const Sched<W>& sc, int t, Item& it,
                                          int bits = 0) {
  const Pattern pat{p.nb, p.g, p.w, p.global_mode};
  const int lane = lane_again(w.lane);
  int list_lo, list_len;
  bool row_global;
  item_coords(p, w, sc, t, it, list_lo, list_len, row_global);
  const int bi = it.bh / p.H, h = it.bh % p.H;
  it.skipped = false;
  it.bits = bits;
  if (kMode >= kOptions && p.skip_q && !block_any_valid_scalar(p.kmask, __builtin_amdgcn_readfirstlane(bi), p.n, __builtin_amdgcn_readfirstlane(it.j))) {
    // the caller reads the mask as a query mask too, and no position of this block is valid:
    // an item without key blocks (O = 0, LSE = -inf)
    it.skipped = true;
    it.partial = 0;
    it.kl = 0;
    it.bh = __builtin_amdgcn_readfirstlane(it.bh);
    it.j = __builtin_amdgcn_readfirstlane(it.j);
    it.chunk = __builtin_amdgcn_readfirstlane(it.chunk);
    it.nchunks = __builtin_amdgcn_readfirstlane(it.nchunks);
    it.slot = __builtin_amdgcn_readfirstlane(it.slot);
    it.cnt = 0;
    return;
  }
  const KeyList kl = item_key_list<kMode != kPlain>(pat, p.rand_idx, p.r, p.kmask, p.n, bi, h, it.j, row_global, list_lo,
                                                    list_len, lane, w.klist, key_bits_of<W>(w.wv, bits));
  it.cnt = kl.cnt;
  it.kl = kl.entry;
  it.partial = kl.partial;
  // all of these are wave uniform; saying so keeps them (and what is computed from them) in
  // scalar registers
  it.bh = __builtin_amdgcn_readfirstlane(it.bh);
  it.j = __builtin_amdgcn_readfirstlane(it.j);
  it.chunk = __builtin_amdgcn_readfirstlane(it.chunk);
  it.nchunks = __builtin_amdgcn_readfirstlane(it.nchunks);
  it.slot = __builtin_amdgcn_readfirstlane(it.slot);
  it.cnt = __builtin_amdgcn_readfirstlane(it.cnt);
  it.partial = __builtin_amdgcn_readfirstlane(it.partial);
}

// First tiles of an item that nobody has fetched ahead.  The query block takes the same road as a
// key block: eight coalesced 1 KB loads into LDS (the V buffer, idle until the first block's V
// arrives), then operand reads.  Register loads of the operand layout would touch every row of
// the tile in each instruction and cost the address unit four times as many cache-line requests.
// Leaves: K(0) in the K buffer, the scaled Q fragments in qb, V(0).t0 as the only load in flight.
template <int W>
__device__ __forceinline__ void fresh_start(const FwdParams& p, const WaveCtx<W>& w, const StraightOffsets& so,
                                            const Item& item, bf16x8 (&qb)[2][4]) {
  const ItemTiles ct(p, item);
  tile_load_async_wave(ct.ktile(0), w.cx.lds_k_a, w.cx.voff);
  tile_load_async_wave(ct.qtile, w.cx.lds_v_a, w.cx.voff);
  wait_tile_loads<0>();
  so.read(w.lds_v, qb);
  wait_lds_reads();
  half_load_async(ct.vtile(0), w.cx.lds_v_a, 0, w.cx.voff);
}

// The two tile streams of an item as global addresses, entry m in lane m (two registers each).
// K stream: the item's K tiles; then, if an item follows, its query tile (twice: the second
// request only rewrites what the first has brought).  V stream: the item's V tiles, then the next
// item's first K tile.  So when an item's last pair is done, its successor's query tile sits in
// the K buffer and its first K tile in the V buffer (the pairs' regular reads take them for K / V
// fragments, which nothing uses).  Without a successor the streams end in the item's first tiles
// again: requests whose data nobody uses, so that every pair issues the same loads and waits for
// the same counts.
struct TileStreams {
  unsigned klo, khi, vlo, vhi;
  __device__ __forceinline__ TileStreams(const FwdParams& p, const Item& it, const Item* next, int lane) {
    const ItemTiles ct(p, it);
    // What the lanes past the item's own tiles hold.  Computed here, with every lane active: these
    // addresses read lane 0 of a list register, which must not happen inside a branch that lane 0
    // does not take (the value of an inactive lane is not defined there).
    unsigned long long k_tail, v_tail;
    if (next) {
      const ItemTiles nx(p, *next);
      k_tail = reinterpret_cast<unsigned long long>(nx.qtile);
      v_tail = reinterpret_cast<unsigned long long>(nx.ktile(0));
    } else {
      k_tail = reinterpret_cast<unsigned long long>(ct.ktile(0));
      v_tail = reinterpret_cast<unsigned long long>(ct.vtile(0));
    }
    const unsigned long long off = static_cast<unsigned long long>(static_cast<unsigned>(it.kl)) << 13;
    const bool own = lane < it.cnt;
    const unsigned long long ka = own ? reinterpret_cast<unsigned long long>(ct.kbase) + off : k_tail;
    const unsigned long long va = own ? reinterpret_cast<unsigned long long>(ct.vbase) + off : v_tail;
    klo = static_cast<unsigned>(ka);
    khi = static_cast<unsigned>(ka >> 32);
    vlo = static_cast<unsigned>(va);
    vhi = static_cast<unsigned>(va >> 32);
  }
  __device__ __forceinline__ const char* k(int m) const {
    return reinterpret_cast<const char*>(
        (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(khi, m))) << 32) |
        static_cast<unsigned>(__builtin_amdgcn_readlane(klo, m)));
  }
  __device__ __forceinline__ const char* v(int m) const {
    return reinterpret_cast<const char*>(
        (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(vhi, m))) << 32) |
        static_cast<unsigned>(__builtin_amdgcn_readlane(vlo, m)));
  }
};

// The same streams without their four vector registers: entries picked by scalar arithmetic, for items with the
// running maximum.
struct ScalarStreams {
  const char* kbase;
  const char* vbase;
  const char* k_tail;
  const char* v_tail;
  int kl, cnt;
  __device__ __forceinline__ ScalarStreams(const FwdParams& p, const Item& it, const Item* next) {
    const ItemTiles ct(p, it);
    kbase = ct.kbase;
    vbase = ct.vbase;
    kl = it.kl;
    cnt = it.cnt;
    if (next) {
      const ItemTiles nx(p, *next);
      k_tail = uniform_ptr(nx.qtile);
      v_tail = uniform_ptr(nx.ktile(0));
    } else {
      k_tail = uniform_ptr(ct.ktile(0));
      v_tail = uniform_ptr(ct.vtile(0));
    }
  }
  __device__ __forceinline__ const char* k(int m) const {
    return m < cnt ? kbase + static_cast<size_t>(__builtin_amdgcn_readlane(kl, m)) * kTile : k_tail;
  }
  __device__ __forceinline__ const char* v(int m) const {
    return m < cnt ? vbase + static_cast<size_t>(__builtin_amdgcn_readlane(kl, m)) * kTile : v_tail;
  }
};

// Operands that nobody reads again, said to the register allocator, which would carry them past the pairs otherwise.
__device__ __forceinline__ void forget(bf16x8 (&f)[2][4]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) asm volatile("" : "=v"(f[t][ks]));
}

// What the first pair of an item "finishes": nothing.
__device__ __forceinline__ void no_predecessor(bf16x8 (&va1)[2][2], bf16x8 (&p3)[2]) {
#pragma unroll
  for (int a = 0; a < 2; ++a) {
#pragma unroll
    for (int e = 0; e < 8; ++e) p3[a][e] = static_cast<__bf16>(0.f);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 8; ++e) va1[a][b][e] = static_cast<__bf16>(0.f);
  }
}

// The block pairs of a single item through the pipeline (a wave's share of a row).  On entry K(0) is in the K buffer
// and V(0).t0 the only load outstanding (fresh_start).
__device__ __forceinline__ void fast_item(const PairCtx& cx, const StraightOffsets& so, const TransposedOffsets& to,
                                          const bf16x8 (&qb)[2][4], bf16x8 (&ka)[2][4], const FwdParams& p,
                                          const Item& item, int lane, f32x16 (&o)[2][2], float (&l_tot)[2]) {
  bf16x8 va[2][2][2], p3[2];
  f32x16 sA;
  const RowSumOperand ones(lane);
  f32x4 ls[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};  // per query tile
  no_predecessor(va[1], p3);
  const int cnt = item.cnt;
  const TileStreams ts(p, item, nullptr, lane);

  // start of the streams: K(0) -> registers, then the loads a pair expects to find outstanding
  read_straight_half(so, cx.lds_k, 0, ka[0]);
  read_straight_half(so, cx.lds_k, 1, ka[1]);
  wait_lds_reads();
  half_load_async(ts.k(1), cx.lds_k_a, 0, cx.voff);
  half_load_async(ts.v(0), cx.lds_v_a, 1, cx.voff);
  wait_tile_loads<8>();
  read_transposed_half(to, cx.lds_v, 0, va[0]);
  unit_scores(ka[0], qb[0], sA);

  for (int i = 0; i < cnt; ++i)
    pair_step(cx, so, to, qb, ka, va, sA, p3, o, ones, ls, ts.k(i + 1), ts.v(i + 1), ts.k(i + 2));
  wait_tile_loads<0>();  // requests past the end of the streams
  // the last unit's share of O and of the row sums
  unit_pv(va[1], p3, o[1], ones, ls[1]);
#pragma unroll
  for (int q = 0; q < 2; ++q) l_tot[q] = row_total(ls[q], lane & 31);
}

template <int kMode>
__device__ __forceinline__ DropRows drop_rows(const FwdParams& p, const Item& item, int lane) {
  DropRows d = {{0u, 0u}, 0u};
  if constexpr (kMode == kDrop) {
    d.thr = drop_pair_threshold(p.drop);
    const uint32_t row0 = static_cast<uint32_t>(item.bh) * static_cast<uint32_t>(p.n) + static_cast<uint32_t>(item.j * kBlk + (lane & 31));
#pragma unroll
    for (int q = 0; q < 2; ++q) d.rk[q] = drop_first(drop_row_key(p.drop, row0 + q * 32));
  }
  return d;
}

// The same with the running maximum, on the same entry.  Leaves the reference exponents (base 2) in m_ref.
// kPeel: the last pair has a body of its own, which requests nothing.  A wave of a short row has one or two pairs, and waiting for
// tiles that nobody uses was a tenth of its time: 12 heads of n = 256, padded inside a block, 7.4 -> 7.15 us, n = 1280 under
// dropout 14.0 -> 13.6.
template <int kMode, int W, bool kPeel>
__device__ __forceinline__ void running_item(const WaveCtx<W>& w, const bf16x8 (&qb)[2][4], bf16x8 (&ka)[2][4], const FwdParams& p,
                                             const Item& item, f32x16 (&o)[2][2], float (&m_ref)[2], float (&l_tot)[2]) {
  const PairCtx& cx = w.cx;
  const LeanOffsets lo(lane_again(w.lane));
  bf16x8 va[2][2][2], p3[2];
  f32x16 s0, s1;
  RowState rs = {{neg_inf(), neg_inf()}, {0.f, 0.f}};
  no_predecessor(va[1], p3);
  zero_acc(o[0]);
  zero_acc(o[1]);
  const DropRows drop = drop_rows<kMode>(p, item, lane_id());
  const int cnt = item.cnt;
  const ScalarStreams ts(p, item, nullptr);

  lo.straight_half(cx.lds_k, 0, ka[0]);
  lo.straight_half(cx.lds_k, 1, ka[1]);
  wait_lds_reads();
  half_load_async(ts.v(0), cx.lds_v_a, 1, cx.voff);
  const bool k_ahead = !kPeel || cnt > 1;
  if (k_ahead) {
    half_load_async(ts.k(1), cx.lds_k_a, 0, cx.voff);
    half_load_async(ts.k(1), cx.lds_k_a, 1, cx.voff);
  }
  unit_scores(ka[0], qb[0], s0);
  unit_scores(ka[1], qb[0], s1);
  for (int i = 0; i < (kPeel ? cnt - 1 : cnt); ++i)
    running_pair<kMode != kPlain, kMode == kDrop>(cx, lo, qb, ka, va, s0, s1, p3, o, rs, drop, drop_words_of<kMode, W>(w.wv),
                                                  __builtin_amdgcn_readlane(item.kl, i), (item.partial >> i) & 1,
                                                  key_bits_of<W>(w.wv, item.bits)[i], ts.k(i + 2), ts.v(i + 1));
  if constexpr (kPeel)
    running_pair<kMode != kPlain, kMode == kDrop, true>(cx, lo, qb, ka, va, s0, s1, p3, o, rs, drop, drop_words_of<kMode, W>(w.wv),
                                                        __builtin_amdgcn_readlane(item.kl, cnt - 1), (item.partial >> (cnt - 1)) & 1,
                                                        key_bits_of<W>(w.wv, item.bits)[cnt - 1], nullptr, nullptr, k_ahead);
  wait_tile_loads<0>();  // requests past the end of the streams
  unit_pv(va[1], p3, o[1]);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    m_ref[q] = rs.m[q];
    l_tot[q] = half_sum(rs.l[q]);
  }
}

// Normalised bf16 output and LSE of a non-global item.  The accumulators hold O^T (a lane owns one
// query and scattered groups of four d); they are turned through LDS (the K buffer) so that global
// memory sees whole rows: 16 bytes per lane, consecutive lanes on consecutive addresses.
template <int W>
__device__ __forceinline__ void store_rows_bf16(const FwdParams& p, const WaveCtx<W>& w, const Item& it,
                                                const f32x16 (&o)[2][2], const float (&inv)[2],
                                                const float (&lse)[2]) {
  const size_t row_blk = static_cast<size_t>(it.bh) * p.n + it.j * kBlk;  // first row of the query block
  const int lane = lane_again(w.lane), hf = lane >> 5, col = lane & 31;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (hf == 0) p.LSE[row_blk + q * 32 + col] = lse[q];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = static_cast<__bf16>(o[q][dt][r4 * 4 + e] * inv[q]);
        // d0 = 32 dt + 8 r4 + 4 hf: 16-byte chunk 4 dt + r4, upper or lower half of it
        *reinterpret_cast<bf16x4*>(w.lds_k + tile_off_bf16(q * 32 + col, dt * 4 + r4) + hf * 8) = v;
      }
  }
  wait_lds_reads();
  __bf16* orow = static_cast<__bf16*>(p.O) + row_blk * kDim;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    u32x4 ov[4];
#pragma unroll
    for (int ii = 0; ii < 4; ++ii)
      ov[ii] = *reinterpret_cast<const u32x4*>(w.lds_k +
                                               tile_off_bf16((half * 4 + ii) * 8 + (lane >> 3), lane & 7));
    wait_lds_reads();  // after the second batch the K buffer may be refilled
#pragma unroll
    for (int ii = 0; ii < 4; ++ii)
      // (non-temporal: the output is not read again, and K and V need the L2: 0.5 us at cfg 2)
      __builtin_nontemporal_store(ov[ii], reinterpret_cast<u32x4*>(orow + ((half * 4 + ii) * 8 + (lane >> 3)) * kDim + (lane & 7) * 8));
  }
}

// Partial triple (reference exponent, row sums, un-normalised O in fp32) of one slice of a row
// that has several, for the merge kernel; O goes through the K buffer in two passes of 32 d.
template <int W>
__device__ __forceinline__ void store_partial(const FwdParams& p, const WaveCtx<W>& w, const Item& it,
                                              const f32x16 (&o)[2][2], const float (&m_ref)[2],
                                              const float (&l_tot)[2]) {
  const int lane = lane_again(w.lane), hf = lane >> 5, col = lane & 31;
  float* pml = p.part_ml + static_cast<size_t>(it.slot) * (2 * kBlk);
  float* po = p.part_o + static_cast<size_t>(it.slot) * (kBlk * kDim);
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (hf == 0) {
      pml[q * 32 + col] = m_ref[q];
      pml[kBlk + q * 32 + col] = l_tot[q];
    }
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[q][dt][r4 * 4 + e];
        *reinterpret_cast<f32x4*>(w.lds_k + tile_off_bf16(q * 32 + col, r4 * 2 + hf)) = v;
      }
    wait_lds_reads();
#pragma unroll
    for (int ii = 0; ii < 8; ++ii) {
      const int row = ii * 8 + (lane >> 3), cc = lane & 7;
      const f32x4 v = *reinterpret_cast<const f32x4*>(w.lds_k + tile_off_bf16(row, cc));
      *reinterpret_cast<f32x4*>(po + row * kDim + dt * 32 + cc * 4) = v;
    }
    wait_lds_reads();
  }
}

// O = 0 and LSE = -inf for the 64 rows of a query block that is not computed (whole rows, 16 bytes
// per lane, straight from registers).
__device__ __forceinline__ void store_zero_rows_bf16(const FwdParams& p, const Item& it) {
  const size_t row_blk = static_cast<size_t>(it.bh) * p.n + it.j * kBlk;
  const int lane = lane_id();
  p.LSE[row_blk + lane] = neg_inf();
  __bf16* orow = static_cast<__bf16*>(p.O) + row_blk * kDim;
  const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int ii = 0; ii < 8; ++ii)
    __builtin_nontemporal_store(z, reinterpret_cast<u32x4*>(orow + (ii * 8 + (lane >> 3)) * kDim + (lane & 7) * 8));
}

// The kernel's argument block as the cold functions below see it.  A reference to the kernel's own
// copy would move that copy, and every later use of it in the hot loop, into scratch memory, and the
// kernel-argument segment pointer is only defined inside the kernel itself.  So the kernel hands its
// segment pointer down and the callee reads the structure again through scalar loads.
typedef const FwdParams __attribute__((address_space(4))) * KernargPtr;

__device__ __forceinline__ FwdParams params_from(const void* kernargs) {
#if defined(__HIP_DEVICE_COMPILE__)
  const char* u = uniform_ptr(static_cast<const char*>(kernargs));
  return *(KernargPtr)(reinterpret_cast<uintptr_t>(u));
#else
  return FwdParams{};
#endif
}

__device__ __forceinline__ const void* kernel_kernargs() {
#if defined(__HIP_DEVICE_COMPILE__)
  return (const void*)(__builtin_amdgcn_kernarg_segment_ptr());
#else
  return nullptr;
#endif
}

// One non-global item with the running maximum, from its first load to its last store: the path of items
// without any key block and of those whose row sums left the safe range of the fixed reference.
template <int kMode, int W>
__device__ __forceinline__ void item_by_recurrence(const FwdParams& p, int t) {
  const WaveCtx<W> w(p.c);
  Sched<W> sc(p, false);
  sc.global_wg = false;  // (a wave of a global-row workgroup that went on to claim other items)
  const StraightOffsets so(w.lane);
  const TransposedOffsets to(w.lane);
  Item it;
  make_item<kMode, W>(p, w, sc, t, it);
  wait_tile_loads<0>();
  bf16x8 qb[2][4], ka[2][4];
  f32x16 o[2][2];
  float m_ref[2] = {neg_inf(), neg_inf()}, l_tot[2] = {0.f, 0.f};
  zero_acc(o[0]);
  zero_acc(o[1]);
  if (it.cnt > 0) {
    fresh_start(p, w, so, it, qb);
    running_item<kMode, W, false>(w, qb, ka, p, it, o, m_ref, l_tot);
  }
  if (it.nchunks == 1) {
    float inv[2], lse[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      inv[q] = l_tot[q] > 0.f ? (kMode == kDrop ? p.drop.rs : 1.f) / l_tot[q] : 0.f;  // (rs: 1, or the dropout scale)
      lse[q] = l_tot[q] > 0.f ? (m_ref[q] + fast_log2(l_tot[q])) * kLn2 : neg_inf();
    }
    store_rows_bf16(p, w, it, o, inv, lse);
  } else {
    store_partial(p, w, it, o, m_ref, l_tot);
  }
}

// The persistent loop's list of such items (lane u of `redo` holds the u-th item), as a called
// function: its registers are not that loop's problem.  One call for the whole list: a call saves
// and restores the callee-saved registers in scratch memory, about 50 KB per wave, which per item
// was most of the time of launches in which many items come here.
template <int kMode, int W>
__device__ __attribute__((noinline)) void redo_items(const void* kernargs, int redo, int n_redo) {
  const FwdParams p = params_from(kernargs);
  for (int u = 0; u < n_redo; ++u) item_by_recurrence<kMode, W>(p, __builtin_amdgcn_readlane(redo, u));
}

// One query block by a whole workgroup: its key list dealt out to the waves (up to 16 key blocks
// each), their (m, l, O~) merged in LDS.  Inlined into the kernel, as the branch taken by the die's first workgroups: a
// real call would start by saving a hundred callee-saved vector registers to scratch memory
// (11 MB of HBM writes per launch at the BERT-base size, measured) for a caller that has nothing
// in them.
template <int kMode, int W, bool kByRow>
__device__ __forceinline__ void global_row_workgroup(const FwdParams& p, const Sched<W>& sc) {
  // (The lane number made once and handed on: with a mask the thread number it comes from is in scratch memory for the
  // sake of the other branch.  64 slices of n = 1536, all keys valid, 26.0 -> 25.4 us.)
  const WaveCtx<W> w(p.c, lane_again(lane_id()));
  const StraightOffsets so(w.lane);
  const TransposedOffsets to(w.lane);
  const int lane = w.lane, wv = w.wv, hf = w.hf, col = w.col;
#ifdef BB_STAMPS
  const long long rt0 = __builtin_amdgcn_s_memrealtime();
#endif
  Item cur;
  make_item<kMode, W>(p, w, sc, 0, cur);
  bool by_recurrence = kMode == kDrop || cur.partial != 0;
  const bool dealt_out = (p.geo.ng == 1 && p.geo.gw_len < kGlobalWaveLen) || sc.row_idx >= p.g * p.geo.ng;
  if ((kMode == kMasked || kMode == kOptions) && dealt_out) {
    // A row with a cut block takes the running maximum in all waves, as the same blocks do in one wave's
    // item.  (Shares of 16 blocks, and of rows of several workgroups: each by itself.)
    if (lane == 0) row_cut<W>()[wv] = by_recurrence;
    __syncthreads();
    int any_cut = 0;
#pragma unroll
    for (int v = 0; v < W; ++v) any_cut |= row_cut<W>()[v];
    by_recurrence = any_cut != 0;
  }
  bf16x8 qb[2][4], ka[2][4];
  f32x16 o[2][2];
  float m_ref[2] = {0.f, 0.f};  // reference exponents (base-2 units); halves agree
  float l_tot[2] = {0.f, 0.f};  // row sums of 2^(s - m_ref)
  zero_acc(o[0]);
  zero_acc(o[1]);
  if (cur.cnt > 0) {
    fresh_start(p, w, so, cur, qb);
    bool bad = by_recurrence;
    if (kMode != kDrop && !bad) {
      fast_item(w.cx, so, to, qb, ka, p, cur, lane, o, l_tot);
#pragma unroll
      for (int q = 0; q < 2; ++q) bad |= !(l_tot[q] >= kSumLo && l_tot[q] <= kSumHi);
      if (__any(bad)) {  // its first tiles again
        const ItemTiles ct(p, cur);
        tile_load_async_wave(ct.ktile(0), w.cx.lds_k_a, w.cx.voff);
        wait_tile_loads<0>();
        half_load_async(ct.vtile(0), w.cx.lds_v_a, 0, w.cx.voff);
      }
    }
    if (__any(bad)) running_item<kMode, W, kByRow>(w, qb, ka, p, cur, o, m_ref, l_tot);
  } else {
    m_ref[0] = m_ref[1] = neg_inf();
  }
  // Un-normalised O of this wave as an fp32 [64 q][64 d] tile in its LDS region: d 0..31 in the
  // first 8 KB, d 32..63 in the second, each laid out like a bf16 tile (128-byte rows of 32 floats).
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[q][dt][r4 * 4 + e];
        *reinterpret_cast<f32x4*>(w.lds_kv + dt * kTile + tile_off_bf16(q * 32 + col, r4 * 2 + hf)) = v;
      }
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (hf == 0) {
      merge_m<W>(wv)[q * 32 + col] = !(l_tot[q] > 0.f) ? neg_inf() : m_ref[q];
      merge_l<W>(wv)[q * 32 + col] = l_tot[q];
    }
#ifdef BB_STAMPS
  if (lane == 0) {  // (nchunks == 1 only: the partial-result area is otherwise in use)
    long long* dst = reinterpret_cast<long long*>(p.part_o) + (static_cast<size_t>(blockIdx.x) * W + wv) * 16;
    dst[0] = rt0;
    dst[1] = __builtin_amdgcn_s_memrealtime();
    dst[2] = -1;
    dst[15] = __builtin_amdgcn_s_getreg((4) | (0 << 6) | (31 << 11));  // HW_ID: where the wave ran
  }
#endif
  __syncthreads();  // all waves of a global workgroup arrive here
  // a wave now owns 64 / W query rows, a lane 64 / W columns of one of them
  constexpr int kCols = kDim / W;
  const size_t row_blk = static_cast<size_t>(cur.bh) * p.n + cur.j * kBlk;
  const int q = wv * kCols + lane / W, part = lane % W;
  float M = neg_inf();
#pragma unroll
  for (int v = 0; v < W; ++v) M = fmaxf(M, merge_m<W>(v)[q]);
  f32x4 acc[kCols / 4];
#pragma unroll
  for (int e = 0; e < kCols / 4; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float L = 0.f;
  if (M != neg_inf()) {
#pragma unroll
    for (int v = 0; v < W; ++v) {
      const float mv = merge_m<W>(v)[q];
      const float wgt = (mv == neg_inf()) ? 0.f : fast_exp2(mv - M);
      L += merge_l<W>(v)[q] * wgt;
#pragma unroll
      for (int e = 0; e < kCols / 4; ++e) {
        const int cc = part * (kCols / 4) + e;
        const f32x4 x = *reinterpret_cast<const f32x4*>(tiles_of<W>(v) + (cc >> 3) * kTile + tile_off_bf16(q, cc & 7));
#pragma unroll
        for (int z = 0; z < 4; ++z) acc[e][z] += x[z] * wgt;
      }
    }
  }
  const size_t row = row_blk + q;
  if (cur.nchunks == 1) {
    const float inv = L > 0.f ? (kMode == kDrop ? p.drop.rs : 1.f) / L : 0.f;  // (rs: 1, or the dropout scale)
    if (part == 0) p.LSE[row] = L > 0.f ? (M + fast_log2(L)) * kLn2 : neg_inf();
    bf16x8* dst = reinterpret_cast<bf16x8*>(static_cast<__bf16*>(p.O) + row * kDim + part * kCols);
#pragma unroll
    for (int e = 0; e < kCols / 8; ++e) {
      bf16x8 v;
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        v[z] = static_cast<__bf16>(acc[2 * e][z] * inv);
        v[4 + z] = static_cast<__bf16>(acc[2 * e + 1][z] * inv);
      }
      dst[e] = v;
    }
  } else {
    // one of several workgroups of a long global row: merged partial triple for the merge kernel
    float* pml = p.part_ml + static_cast<size_t>(cur.slot) * (2 * kBlk);
    if (part == 0) {
      pml[q] = L > 0.f ? M : neg_inf();
      pml[kBlk + q] = L;
    }
    f32x4* dst =
        reinterpret_cast<f32x4*>(p.part_o + static_cast<size_t>(cur.slot) * (kBlk * kDim) + q * kDim + part * kCols);
#pragma unroll
    for (int e = 0; e < kCols / 4; ++e) dst[e] = acc[e];
  }
}

}  // namespace

// The item counters of the dies start every launch at zero (a kernel, not a memset: the call may
// be under graph capture).
__global__ void zero_counters_kernel(int* counters) {
  if (threadIdx.x < kXcd) counters[threadIdx.x * kCounterStride] = 0;
}

// (Eight waves to a row: 12 heads, n = 1024 7.7 -> 8.8 us.)
constexpr int kRowWaves = 4;
// Small launches: a workgroup per row (a kernel of its own, so that the other one keeps its registers
// and schedule).
template <int kMode>
__global__ __launch_bounds__(64 * kRowWaves) __attribute__((amdgpu_waves_per_eu(2)))
void fwd_rows_bf16(FwdParams p) {
  const Sched<kRowWaves> sc(p, true);
  if (sc.row_ok) global_row_workgroup<kMode, kRowWaves, true>(p, sc);
}

template <int kMode, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2)))
void fwd_kernel_bf16(FwdParams p) {
  Sched<W> sc(p, false);
  // dyn: after its first piece of work a wave claims items from its die's counter (zeroed before
  // the launch) instead of taking every wave_stride-th one: with a padding mask items differ in
  // length and some are not computed at all.  The waves of a global-row workgroup then join in
  // when their row is done.
  const bool dyn = kMode == kOptions && p.dyn != 0;
  const bool was_global = sc.global_wg;
  if (sc.global_wg) {
    if (sc.row_ok) global_row_workgroup<kMode, W, false>(p, sc);
    if (!dyn) return;
    __syncthreads();  // the merge has read the other waves' LDS regions; from here on each wave's is its own
    sc.global_wg = false;
  }
  const WaveCtx<W> w(p.c);
  const PairCtx& cx = w.cx;
  const int lane = w.lane;
  char* const lds_k = w.lds_k;
  char* const lds_v = w.lds_v;
  const StraightOffsets so_plain(lane);
  const TransposedOffsets to_plain(lane);
  // (kept in registers where they are all there is to keep)
  auto straight = [&]() { return kMode == kPlain ? so_plain : StraightOffsets(lane_again(lane)); };
  auto transposed = [&]() { return kMode == kPlain ? to_plain : TransposedOffsets(lane_again(lane)); };
  const int n_items_die = sc.n_items_die, wave_stride = sc.wave_stride;
  // the die's next unclaimed item (tickets start after the items the persistent waves begin with)
  auto claim = [&]() {
    int c = 0;
    // Executed in the die's L2, which all claimers of this counter share (a counter per die, a
    // cache line each).  Were two dies ever to work on one counter, each would see its own copy:
    // items done twice with the same result, none left out.
    if (lane == 0)
      c = __hip_atomic_fetch_add(p.counters + sc.xcd * kCounterStride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    c = __builtin_amdgcn_readfirstlane(c);
    // (a counter that has run far past the end must not wrap the sum)
    return c < n_items_die ? wave_stride + c : n_items_die;
  };
  int t_first = static_cast<int>(sc.wg - sc.n_gpart) * W + w.wv;  // first item of this wave
  if (dyn && was_global) t_first = claim();
  const int t_item = __builtin_amdgcn_readfirstlane(t_first);
  if (t_item >= n_items_die) return;

  bf16x8 qb[2][4];  // Q^T operands (B of S^T = K Q^T): lane holds query `col` (+32 for tile B),
                    // d = 16*ks + 8*hf .. +8 -- the "straight" fragments of the Q tile, scaled
  bf16x8 ka[2][4];  // K fragments of the pair in work (they cross the item boundary)
  f32x16 o[2][2];   // [query tile][d tile]: O^T accumulators

#ifdef BB_STAMPS
  // development build (-DBB_STAMPS): per-wave time accounting into the partial-result workspace,
  // 16 x 8 bytes per wave: start and end on the constant 100 MHz clock, items done, shader-clock
  // sums per phase of the persistent loop
  const long long rt0 = __builtin_amdgcn_s_memrealtime();
  long long acc_t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  long long st_t[4] = {0, 0, 0, 0};  // first start in detail: lists, first tiles, operands ready
  long long tprev = __builtin_readcyclecounter();
  int n_done = 0;
#define BB_STAMP(i) do { const long long tn__ = __builtin_readcyclecounter(); acc_t[i] += tn__ - tprev; tprev = tn__; } while (0)
#else
#define BB_STAMP(i)
#endif
  // ---- persistent wave: the die's non-global items t_item, t_item + wave_stride, ...
  // Items with a cut block (and all under dropout) take their pairs with the running maximum.  Items without
  // any key block, and those whose row sums turn out to be outside the safe range, are put on a list and done
  // by item_by_recurrence when the stream has ended (a lane of `redo` each).  Items dealt out: the
  // host sizes the grid so that a wave has at most kListedItems.  Items claimed: a wave with that many
  // on its list takes no more; the one or two it still has in flight find room behind them.
  int redo = 0;       // the list: lane t holds the number of the t-th such item
  int n_redo = 0;
  auto push_redo = [&](int t) {
    if (lane == n_redo) redo = t;
    n_redo = __builtin_amdgcn_readfirstlane(n_redo + 1);
  };
  // the next item at or after t that has a key block (others go to the list); bits: its set of key_bits
  auto next_item = [&](int t, Item& it, int bits) {
    int found = -1;
    while (t < n_items_die) {
      make_item<kMode, W>(p, w, sc, t, it, bits);
      if (it.cnt > 0) {
        found = t;
        break;
      }
      if (kMode >= kOptions && it.skipped && it.nchunks == 1) {  // nothing to compute: its rows are written here
        store_zero_rows_bf16(p, it);
      } else {
        push_redo(t);
      }
      if (dyn) {
        if (n_redo >= kListedItems) break;  // this wave takes no more items, the others do
        t = claim();
      } else {
        t += wave_stride;
      }
    }
    return __builtin_amdgcn_readfirstlane(found);
  };
  // where the search for the item after item t begins
  auto successor = [&](int t) { return dyn ? (n_redo < kListedItems ? claim() : n_items_die) : t + wave_stride; };

  // cur: the item in work; nxt: the one after it (its list is needed before cur's last pairs,
  // which fetch its first tiles); nn: the one after that, built while few loads are in flight.
  // Where the first item's row is does not depend on the pattern table: its query tile is
  // requested (into the K buffer) before anything else, and the table is read under that flight.
  Item cur, nxt, nn;
  {
    int lo_, len_;
    bool rg_;
    item_coords(p, w, sc, t_item, cur, lo_, len_, rg_);
    tile_load_async_wave(query_tile(p, __builtin_amdgcn_readfirstlane(cur.bh), __builtin_amdgcn_readfirstlane(cur.j)),
                         cx.lds_k_a, cx.voff);
  }
  int t_cur = next_item(t_item, cur, 0);
  int t_nxt = -1;
#ifdef BB_STAMPS
  st_t[0] = __builtin_readcyclecounter() - tprev;
#endif
  if (t_cur < 0) wait_tile_loads<0>();  // nothing for the pipelined path: let the request land
  if (t_cur >= 0) {
    // pairs this wave still has to do, roughly (for its issue priority)
    const int pairs_per_item = p.geo.cs > 1 ? kGlobalWaveLen : (p.g + p.w + p.r < kGlobalWaveLen ? p.g + p.w + p.r : kGlobalWaveLen);
    int rem_pairs = dyn ? 0  // (unknown when items are claimed: every wave at the same priority)
                        : __builtin_amdgcn_readfirstlane(((n_items_die - t_cur + wave_stride - 1) / wave_stride) * pairs_per_item);

    // start of the first item.  Skipped items ahead of it: the request above was for another row.
    wait_tile_loads<0>();
    if (t_cur != t_item) {
      tile_load_async_wave(query_tile(p, cur.bh, cur.j), cx.lds_k_a, cx.voff);
      wait_tile_loads<0>();
    }
    straight().read(lds_k, qb);
    wait_lds_reads();
    {
      // K(0) and V(0) together; the next item's list is made while they fly
      const ItemTiles ct(p, cur);
      tile_load_async_wave(ct.ktile(0), cx.lds_k_a, cx.voff);
      const char* v0 = uniform_ptr(ct.vtile(0));
      half_load_async(v0, cx.lds_v_a, 0, cx.voff);
      half_load_async(v0, cx.lds_v_a, 1, cx.voff);
    }
#ifdef BB_STAMPS
    st_t[2] = __builtin_readcyclecounter() - tprev;
#endif
    t_nxt = next_item(successor(t_cur), nxt, 1);  // (scalar loads only, unless there is a padding mask)
    int cnt = __builtin_amdgcn_readfirstlane(cur.cnt);  // pairs of the item in work
#ifdef BB_STAMPS
    st_t[1] = __builtin_readcyclecounter() - tprev;
#endif
    wait_tile_loads<8>();  // K(0)
    straight().read(lds_k, ka);
    wait_lds_reads();
    BB_STAMP(0);

    bool rows_written = false;
    for (;;) {
      bool bad = false;
      float inv[2], lse[2], lsum[2], m_ref[2] = {0.f, 0.f};
      bf16x8 va[2][2][2], p3[2];
      f32x16 sA;
      no_predecessor(va[1], p3);
      // Which kind of pairs: a scalar test (a flag in a vector register was reloaded from scratch memory at the start of every
      // item, with a wait for all that was in flight).  Two ifs and not one with an else: the compiler lays the kinds
      // out one behind the other, and what the second reads lives through the pairs of the first unless it is said
      // not to.  33 and 32 spilled vector registers -> 2 and 7 (kMasked, kOptions; with the lists' lane numbers handed on):
      // 8 sequences of n = 4096, 12 heads, padded at block ends, 61.4 -> 59.0 us, inside blocks 72.1 -> 70.1, 230 global tokens 57.8 -> 55.1.
      unsigned running = kMode == kDrop ? 1u : kMode == kPlain ? 0u : cur.partial;
      if (running != 0) {
        zero_acc(o[0]);
        zero_acc(o[1]);
        const ScalarStreams ts(p, cur, t_nxt >= 0 ? &nxt : nullptr);
        const LeanOffsets lo(lane_again(lane));
        f32x16 s1;
        RowState rs = {{neg_inf(), neg_inf()}, {0.f, 0.f}};
        const DropRows drop = drop_rows<kMode>(p, cur, lane_again(lane));
        half_load_async(ts.k(1), cx.lds_k_a, 0, cx.voff);
        half_load_async(ts.k(1), cx.lds_k_a, 1, cx.voff);
        unit_scores(ka[0], qb[0], sA);
        unit_scores(ka[1], qb[0], s1);
        for (int i = 0; i < cnt;) {
          if ((rem_pairs & 3) == 3 || i == 0) set_issue_priority(rem_pairs);
          running_pair<kMode != kPlain, kMode == kDrop>(cx, lo, qb, ka, va, sA, s1, p3, o, rs, drop, drop_words_of<kMode, W>(w.wv),
                                                        __builtin_amdgcn_readlane(cur.kl, i), (cur.partial >> i) & 1,
                                                        key_bits_of<W>(w.wv, cur.bits)[i], ts.k(i + 2), ts.v(i + 1));
          rem_pairs = __builtin_amdgcn_readfirstlane(rem_pairs - 1);
          i = __builtin_amdgcn_readfirstlane(i + 1);
        }
        BB_STAMP(1);
        unit_pv(va[1], p3, o[1]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float l = half_sum(rs.l[q]);
          m_ref[q] = rs.m[q];
          lsum[q] = l;
          inv[q] = l > 0.f ? (kMode == kDrop ? p.drop.rs : 1.f) / l : 0.f;
          lse[q] = l > 0.f ? (rs.m[q] + fast_log2(l)) * kLn2 : neg_inf();
        }
        forget(ka);
      }
      if constexpr (kMode == kMasked || kMode == kOptions) asm volatile("" : "+s"(running));  // (or the two become one again)
      if (running == 0) {
        zero_acc(o[0]);
        zero_acc(o[1]);
        const StraightOffsets so = straight();
        const TransposedOffsets to = transposed();
        const RowSumOperand ones(lane_again(lane));
        f32x4 ls[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        const TileStreams ts(p, cur, t_nxt >= 0 ? &nxt : nullptr, lane_again(lane));
        half_load_async(ts.k(1), cx.lds_k_a, 0, cx.voff);
        // V(0).t0.  Behind it are V(0).t1, K(1).t0 and the eight 16-byte stores (at least) of rows just written, which
        // it need not wait for (48 slices of n = 3072 31.5 -> 31.2 us, of n = 4096 40.3 -> 40.2; with a mask, where the list builder
        // has waited for them, the branch only costs: 33.0 -> 32.8, all keys valid)
        if (kMode == kPlain && rows_written)
          wait_tile_loads<16>();
        else
          wait_tile_loads<8>();
        read_transposed_half(to, lds_v, 0, va[0]);
        unit_scores(ka[0], qb[0], sA);
        for (int i = 0;;) {
          if ((rem_pairs & 3) == 3 || i == 0) set_issue_priority(rem_pairs);
          pair_step(cx, so, to, qb, ka, va, sA, p3, o, ones, ls, ts.k(i + 1), ts.v(i + 1), ts.k(i + 2));
          rem_pairs = __builtin_amdgcn_readfirstlane(rem_pairs - 1);
          i = __builtin_amdgcn_readfirstlane(i + 1);
          if (__builtin_expect(i >= cnt, 0)) break;  // (the register allocator should favour the pairs)
        }
        // the last unit's share of O, the row sums, the range check
        BB_STAMP(1);
        unit_pv(va[1], p3, o[1], ones, ls[1]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float l = row_total(ls[q], w.col);
          bad |= !(l >= kSumLo && l <= kSumHi);
          lsum[q] = l;
          inv[q] = 1.f / l;
          lse[q] = fast_log2(l) * kLn2;
        }
      }
      // ---- item boundary
      const bool redo_cur = __any(bad);
      if (redo_cur) push_redo(t_cur);

      // the list of the item after the next: here at most four tile loads are in flight, so the
      // waits that building it may need (compiler-placed, for all loads) cost little
      int t_nn = -1;
      BB_STAMP(2);
      if (t_nxt >= 0) {
        t_nn = next_item(successor(t_nxt), nn, cur.bits);  // (cur is done with its bits)
        BB_STAMP(3);
        // The next item's query tile is in the K buffer, its first K tile in the V buffer (the
        // second half may still be landing).  Both go to registers, its first V tile is requested,
        // and this item's output is written under that flight.
        wait_tile_loads<0>();
        const StraightOffsets so = straight();
        so.read(lds_k, qb);
        so.read(lds_v, ka);
        wait_lds_reads();
        const char* v0 = uniform_ptr(ItemTiles(p, nxt).vtile(0));
        half_load_async(v0, cx.lds_v_a, 0, cx.voff);
        half_load_async(v0, cx.lds_v_a, 1, cx.voff);
      }

      BB_STAMP(4);
      if (t_nxt < 0) {
        wait_tile_loads<0>();  // requests past the end of the streams
        // (no instruction: nothing of the last item's operands is kept for a next one)
        forget(qb);
        forget(ka);
      }
      // ---- output, through the K buffer (free now)
      rows_written = !redo_cur && cur.nchunks == 1;
      if (!redo_cur) {
        if (cur.nchunks == 1) {
          store_rows_bf16(p, w, cur, o, inv, lse);
        } else {
          store_partial(p, w, cur, o, m_ref, lsum);
        }
      }
      BB_STAMP(5);
#ifdef BB_STAMPS
      ++n_done;
#endif
      if (t_nxt < 0) break;

      // ---- the next item's stream starts (its K(0) fragments are in registers, V(0) is in flight)
      cur = nxt;
      t_cur = t_nxt;
      nxt = nn;
      t_nxt = t_nn;
      cnt = __builtin_amdgcn_readfirstlane(cur.cnt);
      BB_STAMP(6);
    }
  }
#ifdef BB_STAMPS
  if (lane == 0) {
    long long* dst = reinterpret_cast<long long*>(p.part_o) + (static_cast<size_t>(blockIdx.x) * W + w.wv) * 16;
    dst[0] = rt0;
    dst[1] = __builtin_amdgcn_s_memrealtime();
    dst[2] = n_done;
    for (int i = 0; i < 7; ++i) dst[3 + i] = acc_t[i];
    dst[10] = st_t[0];
    dst[11] = st_t[1];
    dst[12] = st_t[2];
    dst[15] = __builtin_amdgcn_s_getreg((4) | (0 << 6) | (31 << 11));  // HW_ID: where the wave ran
  }
#endif

  // ---- the listed items, by the classical recurrence
  if (n_redo > 0) redo_items<kMode, W>(kernel_kernargs(), redo, n_redo);
}

int launch_fwd_bf16_main(const FwdParams& p, hipStream_t stream) {
  const unsigned grid = p.geo.by_row ? DieItems(p.BH, p.geo.g_wgs).grid()
                                     : static_cast<unsigned>(kXcd) * (p.geo.bh_rounds * p.geo.g_wgs + p.geo.p_wgs);
  if (grid == 0) return BB_OK;
  if (p.dyn) {
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, stream, p.counters);
    if (hipGetLastError() != hipSuccess) return BB_ERR_LAUNCH;
  }
  const int mode = p.drop.thr != 0 ? kDrop : p.skip_q ? kOptions : p.kmask ? kMasked : kPlain;
  static constexpr void (*kRows[4])(FwdParams) = {fwd_rows_bf16<kPlain>, fwd_rows_bf16<kMasked>, fwd_rows_bf16<kOptions>, fwd_rows_bf16<kDrop>};
  static constexpr void (*kItems[2][4])(FwdParams) = {
      {fwd_kernel_bf16<kPlain, 4>, fwd_kernel_bf16<kMasked, 4>, fwd_kernel_bf16<kOptions, 4>, fwd_kernel_bf16<kDrop, 4>},
      {fwd_kernel_bf16<kPlain, 8>, fwd_kernel_bf16<kMasked, 8>, fwd_kernel_bf16<kOptions, 8>, fwd_kernel_bf16<kDrop, 8>}};
  const auto kernel = p.geo.by_row ? kRows[mode] : kItems[p.geo.waves == 8][mode];
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * p.geo.waves), 0, stream, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    fprintf(stderr, "bigbird: launch of fwd_kernel_bf16 failed: %s\n", hipGetErrorString(e));
    return BB_ERR_LAUNCH;
  }
  return BB_OK;
}

}  // namespace bb
