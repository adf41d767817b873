// Pieces of the fp32 kernels of small launches.  A workgroup owns eight positions of one block (queries, or keys
// in the dK/dV kernel) and deals the block's list out to its eight waves; their results meet in LDS, so that no
// launch follows that adds up partial results.
//
// All products run on v_mfma_f32_4x4x1_16b_f32 (16 independent 4x4 products of one contraction step each, at the rate of the
// larger fp32 forms).  With lane = 16 g + 4 a + t:
//   row form of a 64 x 64 tile X: X[16 kt + 4 a + t][16 u + 4 g ..+3], the A operand of a product over d in which group g
//     takes the d with (d / 4) % 4 = g;
//   own positions Y (four to an operand): Y[t][16 u + 4 g ..+3], its B operand;
//   the accumulator's four elements are then rows 16 kt + 4 a + 0..3 against position t, each group's share of the
//     sum over d.  sum_over_groups adds the groups and leaves row 16 kt + 4 a + g in the lane: 64 x 4 values in four
//     registers;
//   these are, as they stand, the A operand of the product over the tile's rows (broadcast inside each group, so
//     that group g takes the rows with row % 4 = g): position i = 0..3 in element i, B operand X[4 s + g][4 m ..+3] with
//     m = lane % 16, whole rows at a time.  Element i of accumulator e: position i, column 4 m + e, group g's share.
// Tiles reach LDS sixteen rows at a time (quarters), straight from global memory; 16-byte chunk c of row r is at
// position c ^ (r % 16) of its row, so that both forms are read without bank conflicts.  (Row form straight from global
// memory touches four rows with every four lanes: four times the cycles of the address unit, which was all the
// time there was.)
#ifndef BB_F32_ROWS_H_
#define BB_F32_ROWS_H_

#include "key_list.h"
#include "tile_ops.h"

#include <type_traits>
#include "kernel_common.h"

namespace bb {

constexpr int kOwn = 8;            // positions of a workgroup
constexpr int kRowsWavesF32 = 8;   // waves that share a list
constexpr int kRowsThreadsF32 = 64 * kRowsWavesF32;
constexpr int kOwnTiles = kBlk / kOwn;
constexpr int kQuarterF32 = 16 * kDim * 4;  // bytes of sixteen rows
constexpr int kQuarterLoads = 4;            // vector memory instructions that bring them

struct RowsLane {
  int g, a, t, m;
  __device__ __forceinline__ explicit RowsLane(int lane) : g(lane >> 4), a((lane >> 2) & 3), t(lane & 3), m(lane & 15) {}
  __device__ __forceinline__ int row(int kt) const { return 16 * kt + 4 * a + g; }  // of a summed score
};

// Sum of x over the four groups for each of its elements; group g is left with element g.
__device__ __forceinline__ float sum_over_groups(const f32x4& x) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[0]), __float_as_uint(x[2]), false, false);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[1]), __float_as_uint(x[3]), false, false);
  const float even = __uint_as_float(p[0]) + __uint_as_float(p[1]);  // groups 0, 1: element 0; 2, 3: element 2
  const float odd = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(even), __float_as_uint(odd), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// x combined over the 16 lanes with the same t, in all of them.
template <class Op>
__device__ __forceinline__ float over_rows(float x, Op op) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(q[0]), __uint_as_float(q[1]));
  x = op(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, true)));  // row_ror:4
  return op(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, true)));  // row_ror:8
}
__device__ __forceinline__ float add_over_rows(float x) { return over_rows(x, [](float p, float q) { return p + q; }); }
__device__ __forceinline__ float max_over_rows(float x) { return over_rows(x, [](float p, float q) { return fmaxf(p, q); }); }

// Sum over the four groups alone.
__device__ __forceinline__ float add_over_groups(float x) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// The value of position i (lane t = i of each quad), in all lanes of the quad.
template <int I>
__device__ __forceinline__ float of_position(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), I * 0x55, 0xf, 0xf, true));
}

// The eight own rows (first one at `rows`).
__device__ __forceinline__ void own_rows(const float* rows, const RowsLane& l, f32x4 (&y)[2][4]) {
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int u = 0; u < 4; ++u) y[q][u] = *reinterpret_cast<const f32x4*>(rows + (4 * q + l.t) * kDim + 16 * u + 4 * l.g);
}

// Sixteen rows, global -> LDS, by one wave: instruction q fills rows 4 q ..+3 linearly and fetches for each place the
// chunk that belongs there.  Invisible to the compiler's wait counts, like half_load_async.
struct QuarterLoads {
  unsigned voff[4];
  __device__ __forceinline__ explicit QuarterLoads(int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q) voff[q] = (lane >> 4) * 256 + (((lane & 15) ^ (4 * q + (lane >> 4))) << 4);
  }
  __device__ __forceinline__ void request(const float* rows, unsigned lds) const {
    const char* g = uniform_ptr(reinterpret_cast<const char*>(rows));
    asm volatile(
        "s_mov_b32 m0, %5\n\t"
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %0, %4\n\t"
        "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
        "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
        "global_load_lds_dwordx4 %3, %4 offset:3072"
        :
        : "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(g), "s"(__builtin_amdgcn_readfirstlane(lds))
        : "memory");
  }
};

// Both forms of a quarter in LDS.
struct QuarterForms {
  int row, column;
  __device__ __forceinline__ explicit QuarterForms(const RowsLane& l)
      : row((4 * l.a + l.t) * 256 + ((l.g ^ (4 * l.a + l.t)) << 4)), column(l.g * 256 + ((l.m ^ l.g) << 4)) {}
  __device__ __forceinline__ void row_form(const char* quarter, f32x4 (&x)[4]) const {
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const f32x4*>(quarter + (row ^ (u << 6)));
  }
  __device__ __forceinline__ void column_form(const char* quarter, f32x4 (&z)[4]) const {
#pragma unroll
    for (int s = 0; s < 4; ++s) z[s] = *reinterpret_cast<const f32x4*>(quarter + (column ^ (s << 6)) + s * 1024);
  }
};

// Products of two sets of sixteen rows with own rows, side by side (four chains of matrix instructions: one chain waits
// for itself): s[q] is row l.row(kt) of a set against position 4 q + t.
__device__ __forceinline__ void row_products(const f32x4 (&x0)[4], const f32x4 (&y0)[2][4], float (&s0)[2],
                                             const f32x4 (&x1)[4], const f32x4 (&y1)[2][4], float (&s1)[2]) {
  f32x4 a0[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, a1[2] = {a0[0], a0[0]};
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int q = 0; q < 2; ++q) a0[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(x0[u][e], y0[q][u][e], a0[q], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 2; ++q) a1[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(x1[u][e], y1[q][u][e], a1[q], 0, 0, 0);
    }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    s0[q] = sum_over_groups(a0[q]);
    s1[q] = sum_over_groups(a1[q]);
  }
}

// acc[q][e] += P^T X over sixteen rows in column form: P as row_products leaves it.
__device__ __forceinline__ void add_rows(const f32x4 (&z)[4], const float (&p)[2], f32x4 (&acc)[2][4]) {
  auto step = [&](auto S) {
    constexpr int k = decltype(S)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[q][e] = __builtin_amdgcn_mfma_f32_4x4x1f32(p[q], z[k][e], acc[q][e], 2, k, 0);
  };
  step(std::integral_constant<int, 0>{});
  step(std::integral_constant<int, 1>{});
  step(std::integral_constant<int, 2>{});
  step(std::integral_constant<int, 3>{});
}

// A wave's accumulators, groups added, as rows of 64 floats.
__device__ __forceinline__ void store_own(float (*dst)[kDim], const RowsLane& l, const f32x4 (&acc)[2][4]) {
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      dst[4 * q + i][4 * l.m + l.g] = sum_over_groups(f32x4{acc[q][0][i], acc[q][1][i], acc[q][2][i], acc[q][3][i]});
}

__device__ __forceinline__ void clear_own(f32x4 (&acc)[2][4]) {
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[q][e] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Validity of this lane's row of quarter kt, from a block's validity bits.
__device__ __forceinline__ bool row_valid(const uint32_t* bits, const RowsLane& l, int kt) {
  return (bits[kt >> 1] >> (l.row(kt) & 31)) & 1;
}

// Workgroup id -> slice, block (global ones first) and eight of its positions.  The positions vary slowest, so
// that the long lists of global blocks are spread over the dies also where a slice is cut into runs.
struct OwnItem {
  int bh, j, first;  // first: of the eight positions, inside the block
  bool global;
};
__device__ __forceinline__ bool decode_own(const Pattern& pat, int BH, unsigned wg, OwnItem* it) {
  int item;
  if (!DieItems(BH, pat.nb * kOwnTiles).decode(wg, &it->bh, &item)) return false;
  const int rank = item % pat.nb;
  it->first = item / pat.nb * kOwn;
  it->global = rank < pat.g;
  it->j = it->global ? pat.global_block(rank) : pat.sparse_block(rank - pat.g);
  return true;
}
inline unsigned own_grid(int BH, int nb) { return DieItems(BH, nb * kOwnTiles).grid(); }

// Where these kernels run: launches of up to a workgroup per compute unit (a unit holds one: its waves' tiles in LDS) and
// lists of up to two entries a wave.  Forward / whole step in us, slices of the list with partial results added by
// launches of their own against these: 2 slices of n = 1024: 15.7 / 63.4 and 11.8 / 46.1; 4 of n = 512: 25.7 / 57.0
// and 9.0 / 35.3; 3 of n = 640: 12.8 / 48.9 and 11.5 / 43.0.  What bounds them is the matrix rate of the compute units that own
// global blocks (two entries a wave there, 2 us each) on top of 6 us for launch, list, first tile and merge.  With two
// workgroups to a unit: 4 of n = 1024 19.6 / 82.0 and 19.2 / 82.0, 4 of n = 768 17.1 / 70.1 and 18.9 / 74.7.  One slice of 13 to 16
// blocks fits the chip in slices of one pair: 11.7 / 44.3 and 11.7 / 45.8.  One of n = 1280 (three entries): 13.0 / 47.8 and 15.2 / 55.5.
inline bool rows_f32_bwd(int BH, int nb) {
  const long long blocks = static_cast<long long>(BH) * nb;
  return blocks <= 32 && nb <= 2 * kRowsWavesF32 && (nb <= 12 || blocks > 16);
}
// A forward of up to eight blocks cuts no list (it needs no workspace): 3 us for every block in series there, while a
// round of these workgroups takes 7 to 8 us (12 slices of n = 512: 25.8 and 23.9; 24 of n = 256: 14.8 and 18.4).  What counts
// is the longest list there is: without global blocks n = 512 has lists of 6 (12 slices: 20.5 and 23.5), and under a mask
// they may be shorter (12 of n = 512, padded: 24.8 and 26.4).  A single block has nothing to deal out (plain 6.4 and 6.2 us,
// masked 7.3 and 7.4, masked with dropout 7.5 and 8.0).  Past eight blocks the other kernel cuts lists for several waves, and
// here a wave's share is two entries, which take longest under dropout (one slice of n = 640: 11.7 and 12.9, without dropout 11.5
// and 11.5, padded 12.1 and 9.4; two of n = 768, dropout: 12.6 and 13.1, n = 1024: 16.4 and 13.3).
inline bool rows_f32_fwd(int BH, int nb, int g, int w, int r, bool masked, bool drop) {
  const long long blocks = static_cast<long long>(BH) * nb;
  const int longest = g > 0 ? nb : longest_sparse_list(nb, g, w, r);
  if (nb == 1) return !drop && blocks <= 32;
  if (drop && !masked && longest > kRowsWavesF32 + 1 && blocks <= 30) return false;
  return rows_f32_bwd(BH, nb) || (nb <= kChunkGlobal && blocks <= (longest == 8 && !masked ? 96 : longest >= 6 ? 64 : 32));
}

// This wave's share of a query block's key-block list.
__device__ __forceinline__ KeyList own_key_list(const Pattern& pat, const int32_t* rand_idx, int r, const uint8_t* kmask, int n,
                                                int bi, int h, const OwnItem& it, int wv, int lane, int* klist, uint32_t (*key_bits)[2]) {
  const int most = it.global ? pat.nb : (pat.g + pat.w + r < pat.nb ? pat.g + pat.w + r : pat.nb);
  const int share = (most + kRowsWavesF32 - 1) / kRowsWavesF32;
  return item_key_list<true>(pat, rand_idx, r, kmask, n, bi, h, it.j, it.global, wv * share, share, lane, klist, key_bits);
}

}  // namespace bb
#endif  // BB_F32_ROWS_H_
