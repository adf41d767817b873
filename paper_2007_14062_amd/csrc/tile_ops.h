// Asynchronous tile staging and synchronisation pieces shared by the bf16 kernels.
#ifndef BB_TILE_OPS_H_
#define BB_TILE_OPS_H_

#include "kernel_common.h"

namespace bb {

constexpr int kTile = kBlk * kDim * 2;  // one 64x64 bf16 tile: 8 KB
constexpr int kHalfTile = kTile / 2;    // 32 rows

// s_waitcnt immediate that waits for all but `n` vector-memory loads (gfx9 encoding:
// vmcnt in bits 3:0 and 15:14, other counters left at their maxima).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int kLgkmcnt0 = 15 | (3 << 14) | (7 << 4);  // wait for all LDS reads, nothing else

__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uintptr_t v = reinterpret_cast<uintptr_t>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v));
  const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v >> 32));
  return reinterpret_cast<const char*>((static_cast<uintptr_t>(hi) << 32) | lo);
}

// Per-lane byte offsets of half_load_async.
__device__ __forceinline__ void half_load_offsets(int lane, unsigned (&voff)[2]) {
#pragma unroll
  for (int par = 0; par < 2; ++par)
    voff[par] = (lane >> 3) * 128 + (((lane & 7) ^ tile_swizzle(par * 8 + (lane >> 3))) << 4);
}

// Half of a 64x64 bf16 tile (rows 32*hh .. +32), global -> LDS, by one wave: four
// instructions of 64 lanes x 16 bytes.  Instruction ii fills LDS rows 8*ii .. 8*ii+7 of
// the half linearly (lane l lands on row l/8, chunk position l%8) and fetches, for that
// place, the chunk the swizzle stores there.  The swizzle depends on row bits 1..3, i.e. on
// l/8 and on the parity of ii: voff[0] / voff[1] are the per-lane byte offsets for even /
// odd ii.  The instruction's immediate offset moves the global and the LDS address alike,
// so the four instructions share one base pair (M0, scalar address).
// Written as inline asm so that the compiler's wait-count bookkeeping does not see
// these loads: it would otherwise drain them before every LDS read.  The waits
// are placed by hand (loads return in order, so vmcnt(N) is exact).
__device__ __forceinline__ void half_load_async(const char* gtile_, unsigned lds, int hh,
                                                const unsigned (&voff)[2]) {
  const char* gtile = uniform_ptr(gtile_);  // wave uniform by construction: it has to sit in scalar registers
  asm volatile(
      "s_mov_b32 m0, %3\n\t"
      "s_nop 4\n\t"  // wait states the compiler cannot see to from outside: M0 written by a scalar instruction (1) and an
                       // address register pair that a vector instruction (v_readlane) may just have written (5)
      "global_load_lds_dwordx4 %0, %2\n\t"
      "global_load_lds_dwordx4 %1, %2 offset:1024\n\t"
      "global_load_lds_dwordx4 %0, %2 offset:2048\n\t"
      "global_load_lds_dwordx4 %1, %2 offset:3072"
      :
      : "v"(voff[0]), "v"(voff[1]), "s"(gtile + hh * kHalfTile), "s"(lds + hh * kHalfTile)
      : "memory");  // M0 is written here; it is a reserved register that the compiler only sets right before
                    // instructions of its own that read it, and this kernel has none
}

__device__ __forceinline__ void tile_load_async_wave(const char* gtile_, unsigned lds, const unsigned (&voff)[2]) {
  const char* gtile = uniform_ptr(gtile_);  // wave-uniform by construction: keep it in scalar registers
  half_load_async(gtile, lds, 0, voff);
  half_load_async(gtile, lds, 1, voff);
}

// Waits and compiler fences.  The tile loads are invisible to the compiler's wait-count
// bookkeeping (inline asm), so every wait for them is written out; loads return in order,
// which makes "all but the N youngest" exact.
template <int N>
__device__ __forceinline__ void wait_tile_loads() {
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(N));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds_reads() {
  __builtin_amdgcn_s_waitcnt(kLgkmcnt0);
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return static_cast<unsigned>(reinterpret_cast<uintptr_t>((BB_LDS const char*)(p)));
}


// Enqueue one 256-byte vector (64 floats): global -> LDS, 4 bytes per lane, lane l
// lands at lds + 4*l.  `gvec` is the wave-uniform address of the vector.
__device__ __forceinline__ void vec_load_async(const float* gvec, unsigned lds, unsigned lane) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 4\n\t"
      "global_load_lds_dword %0, %1"
      :
      : "v"(lane * 4u), "s"(gvec), "s"(lds)
      : "memory");
}

// MFMA operand fragments of a 64x64 bf16 tile held in LDS (128-byte rows, swizzled
// chunks).  "Straight": the tile's rows are the MFMA's non-contracted index and its
// columns (d) the contraction: fragment [t][ks] = row 32t + lane%32, columns
// 16ks + 8*(lane/32) .. +8.  Used for K in S^T = K Q^T, for V in dP^T = V dO^T, for Q
// and dO in the key-major backward kernel.
struct StraightOffsets {
  int off[4];  // byte offsets for ks = 0..3 of row lane%32 (t adds 4096)
  __device__ __forceinline__ explicit StraightOffsets(int lane) {
    const int col = lane & 31, hf = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) off[ks] = tile_off_bf16(col, ks * 2 + hf);
  }
  __device__ __forceinline__ void read(const char* tile, bf16x8 (&f)[2][4]) const {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        f[t][ks] = *reinterpret_cast<const bf16x8*>(tile + off[ks] + t * 4096);
  }
};

// "Transposed": the tile's rows are the contraction index, taken in the order the
// 32x32 accumulator layout hands them over: fragment [dt][sg] belongs to output row
// (tile column) 32dt + lane%32 and holds, in contraction slot 8*(lane/32) + kk, tile
// row 16sg + 4*(lane/32) + kk (kk < 4) or 16sg + 8 + 4*(lane/32) + kk - 4.  Read with
// ds_read_b64_tr_b16.  Used for V^T in O^T += V^T P^T, K^T in dQ^T += K^T dS^T, dO^T and
// Q^T in the key-major backward kernel.
struct TransposedOffsets {
  int off[2][2];  // byte offsets for dt = 0, 1 and the two 4-row pieces (sg adds 2048)
  __device__ __forceinline__ explicit TransposedOffsets(int lane) {
    const int hf = lane >> 5, gq = lane >> 4, li = lane & 15;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        off[dt][half] = tile_off_bf16(half * 8 + hf * 4 + (li >> 2), dt * 4 + (gq & 1) * 2 + ((li & 3) >> 1)) +
                        (li & 1) * 8;
  }
  __device__ __forceinline__ bf16x8 read_one(const char* tile, int dt, int sg) const {
    // rows 16*sg + {0, 8} + (4*hf + li/4): adding a multiple of 16 rows keeps the swizzle
    const s16x4 lo = lds_read_tr16(tile + off[dt][0] + sg * 2048);
    const s16x4 hi = lds_read_tr16(tile + off[dt][1] + sg * 2048);
    union { struct { s16x4 a, b; } h2; bf16x8 v; } u;
    u.h2.a = lo;
    u.h2.b = hi;
    return u.v;
  }
};

// One half (32 rows) of either kind, by one wave.
__device__ __forceinline__ void read_straight_half(const StraightOffsets& so, const char* tile, int t, bf16x8 (&f)[4]) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) f[ks] = *reinterpret_cast<const bf16x8*>(tile + so.off[ks] + t * kHalfTile);
}

__device__ __forceinline__ void read_transposed_half(const TransposedOffsets& to, const char* tile, int t,
                                            bf16x8 (&f)[2][2]) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int sgl = 0; sgl < 2; ++sgl) f[dt][sgl] = to.read_one(tile, dt, 2 * t + sgl);
}

// Padded keys of a unit (32 keys x 32 queries, a lane per query) leave its packed dS values here: after the
// conversion and before the product with K, whose rows have to be finite, sees them (the values may be anything, also
// not a number).  bits: validity of the 32 keys of the unit, in key order.  Element kk of operand sgl belongs to key
// 16 sgl + 8 (kk / 4) + 4 hf + kk % 4 (acc_row).  Three instructions per packed pair on the vector port --
// only block pairs with padded keys inside pay them: the others take one scalar branch per unit.
__device__ __forceinline__ void drop_padded_keys(uint32_t bits, int hf, bf16x8 (&pb)[2]) {
  const int b = static_cast<int>(bits >> (4 * hf));
#pragma unroll
  for (int sgl = 0; sgl < 2; ++sgl) {
    union { bf16x8 v; uint32_t d[4]; } u;
    u.v = pb[sgl];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int key = acc_row(sgl * 8 + 2 * m, 0);
      const uint32_t even = static_cast<uint32_t>(__builtin_amdgcn_sbfe(b, key, 1));      // 0 or ~0
      const uint32_t odd = static_cast<uint32_t>(__builtin_amdgcn_sbfe(b, key + 1, 1));
      u.d[m] &= (even & 0xffffu) | (odd & 0xffff0000u);
    }
    pb[sgl] = u.v;
  }
}

}  // namespace bb

// Workgroup barrier without the memory fence of __syncthreads(): the fence would
// drain the LDS-bound loads still in flight.  Ordering is kept by the explicit
// counter waits next to each use; the empty asm stops compiler reordering.
#define BB_BARRIER()                       \
  do {                                     \
    asm volatile("" ::: "memory");         \
    __builtin_amdgcn_s_barrier();          \
    asm volatile("" ::: "memory");         \
  } while (0)


#endif  // BB_TILE_OPS_H_
