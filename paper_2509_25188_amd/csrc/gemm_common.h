// Device helpers shared by the bf16 GEMM kernels (many rows: gemm_bf16.hip, few rows: gemm_few_rows.hip).
#pragma once
#include "common.h"

#include <type_traits>

namespace l2pd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// fp32 -> bf16, round to nearest even, two values per v_cvt_pk_bf16_f32; lo lands in bits 15:0
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ unsigned short f2bf(float f) { return (unsigned short)(pack_bf16(f, 0.f) & 0xffffu); }

// Lane exchange inside a row of 16 lanes by DPP (no LDS): quad_perm for xor 1 / xor 2, row_ror for rotations.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor = 0x120;
template <int CTRL>
__device__ __forceinline__ unsigned dpp(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float dppf(float x) {
  return __builtin_bit_cast(float, dpp<CTRL>(__builtin_bit_cast(unsigned, x)));
}

// 4x4 transpose inside every aligned group of four lanes: on entry lane j of a group holds
// element (j, k) in w[k]; on return it holds element (k, j).  In the MFMA C layout a lane owns one
// column and four consecutive rows, so the transpose gives each lane four consecutive columns of
// one row, which it can store as one piece instead of four.
__device__ __forceinline__ void quad_transpose(unsigned (&w)[4], int lane) {
  const bool o1 = lane & 1, o2 = lane & 2;
  unsigned s0 = o1 ? w[0] : w[1], s1 = o1 ? w[2] : w[3];
  s0 = dpp<kDppXor1>(s0);
  s1 = dpp<kDppXor1>(s1);
  if (o1) { w[0] = s0; w[2] = s1; } else { w[1] = s0; w[3] = s1; }
  unsigned t0 = o2 ? w[0] : w[2], t1 = o2 ? w[1] : w[3];
  t0 = dpp<kDppXor2>(t0);
  t1 = dpp<kDppXor2>(t1);
  if (o2) { w[0] = t0; w[1] = t1; } else { w[2] = t0; w[3] = t1; }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {   // s_waitcnt vmcnt(N) only (expcnt / lgkmcnt untouched)
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// Workgroup barrier without the memory-model fence of __syncthreads(), which would wait for every
// outstanding global load (vmcnt(0)) and so drain the prefetch ring.  LDS visibility is ordered by
// the explicit waits around it; the empty asm statements keep the compiler from moving LDS
// accesses across the barrier.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// 16 bytes per lane, global -> LDS without passing through VGPRs.  The LDS destination of the whole
// wavefront is M0 + 16 * lane.  Written as inline asm on purpose: the compiler's wait-count pass
// falls back to lgkmcnt(0) before every LDS read while a direct-to-LDS load it knows of is in
// flight, which would serialise the fragment prefetch; completion is tracked by hand with
// wait_vmcnt<>().  (Untracked extra loads can only make the compiler's own vmcnt waits stricter,
// because vmcnt retires in order.)
__device__ __forceinline__ void dma16(const void* gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gptr), "s"(lds_addr)
               : "memory", "m0");
}

// The same for weights that come from memory once and are not wanted again before the cache has forgotten them (Gate::cold).
// Rows of 8 KB in pieces of 128 bytes, loads alone (an order of their own, no bound for a product): 201 MB 34.2 us against 37.1,
// 1,036 MB 159 against 174.  Weights that stay in the
// memory-side cache (256 MB) from pass to pass lose by it: 201 MB again and again 35.3 against 30.7.
__device__ __forceinline__ void dma16_once(const void* gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
               :
               : "v"(gptr), "s"(lds_addr)
               : "memory", "m0");
}
template <bool COLD>
__device__ __forceinline__ void dma16_weights(const void* gptr, unsigned lds_addr) {
  if constexpr (COLD) dma16_once(gptr, lds_addr);
  else dma16(gptr, lds_addr);
}

// Tiles of a launch: consecutive ids on one XCD share a weight panel (eight row tiles of it, then the next eight).
struct TileMap {
  int tiles_m, tiles_n, total, per_xcd;
  Div per_split, chunk, last;   // by tiles_m * tiles_n, by 8 * tiles_n, by the row tiles of the last chunk
  int per_split_n;
  TileMap() {}
  TileMap(int tm, int tn, int splits)
      : tiles_m(tm), tiles_n(tn), total(tm * tn * splits), per_xcd((tm * tn * splits + 7) / 8), per_split(tm * tn),
        chunk(8 * tn), last(tm % 8 ? tm % 8 : 8), per_split_n(tm * tn) {}
  // false: no tile for this workgroup
  __device__ __forceinline__ bool place(int block, int* z, int* tile_m, int* tile_n) const {
    const int v = (block & 7) * per_xcd + (block >> 3);
    if (v >= total) return false;
    *z = per_split(v);
    int rem = v - *z * per_split_n;
    const int c = chunk(rem);
    rem -= c * 8 * tiles_n;
    const int n = min(8, tiles_m - c * 8);    // row tiles of the chunk
    const int part = last(rem);
    *tile_n = n == 8 ? rem >> 3 : part;
    *tile_m = c * 8 + rem - *tile_n * n;
    return true;
  }
};

}  // namespace l2pd
