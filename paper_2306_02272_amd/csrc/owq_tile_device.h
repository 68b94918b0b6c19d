// Device-side pieces shared by the kernels of the tile layout: operand types of the
// 32x32x16 fp16 matrix instruction, the place of every pair of codes inside its 16-bit
// window, and the A operand made straight from a lane's dwords of codes.
#pragma once
#include <hip/hip_runtime.h>

#include "owq_device.h"

namespace owq {

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f16_t __attribute__((ext_vector_type(16)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));

constexpr int kUnitsPerTile = 2048;   // 16-byte units of one staged activation tile (256 columns x 64 tokens)

// Bit offset o of pair i (columns 2i, 2i+1) of octet t of a block inside its 16-bit window;
// the pair is OR-ed into 2^(10-o).  3-bit: the octet's place in its quad of 32 codes decides.
__device__ __forceinline__ constexpr int pair_offset(int bits, int t, int i) {
  constexpr int off3[4][4] = {{0, 3, 6, 1}, {4, 7, 2, 5}, {0, 3, 6, 1}, {4, 7, 4, 7}};
  constexpr int off4[4] = {0, 4, 2, 6};
  return bits == 3 ? off3[t & 3][i] : off4[i];
}

// A operand of k-step S (16 columns) from the lane's dwords: four packed pairs 2^(10-o)+q.
template <int BITS, int S>
__device__ __forceinline__ h8_t a_operand(const u32 *wd, const Magic &M) {
  u32 r0, r1, r2, r3;
  if (BITS == 3) {
    constexpr int u = S >> 2, o = S & 3;
    const u32 d0 = wd[3 * u], d1 = wd[3 * u + 1], d2 = wd[3 * u + 2];
    if (o == 0) {
      const u32 w1 = __builtin_amdgcn_perm(d1, d0, 0x06030401u);
      r0 = andor(d0, field(3, 0), M.m[0]); r1 = andor(d0, field(3, 3), M.m[3]);
      r2 = andor(d0, field(3, 6), M.m[6]); r3 = andor(w1, field(3, 1), M.m[1]);
    } else if (o == 1) {
      const u32 w1 = __builtin_amdgcn_perm(d1, d0, 0x06030401u);
      r0 = andor(w1, field(3, 4), M.m[4]); r1 = andor(w1, field(3, 7), M.m[7]);
      r2 = andor(d1, field(3, 2), M.m[2]); r3 = andor(d1, field(3, 5), M.m[5]);
    } else if (o == 2) {
      const u32 w3 = __builtin_amdgcn_perm(d2, d1, 0x06030401u);
      r0 = andor(w3, field(3, 0), M.m[0]); r1 = andor(w3, field(3, 3), M.m[3]);
      r2 = andor(w3, field(3, 6), M.m[6]); r3 = andor(d2, field(3, 1), M.m[1]);
    } else {
      const u32 w5 = d2 >> 6;
      r0 = andor(d2, field(3, 4), M.m[4]); r1 = andor(d2, field(3, 7), M.m[7]);
      r2 = andor(w5, field(3, 4), M.m[4]); r3 = andor(w5, field(3, 7), M.m[7]);
    }
  } else {
    const u32 d = wd[S], w = d >> 6;
    r0 = andor(d, field(4, 0), M.m[0]); r1 = andor(d, field(4, 4), M.m[4]);
    r2 = andor(w, field(4, 2), M.m[2]); r3 = andor(w, field(4, 6), M.m[6]);
  }
  const u32x4 v = {r0, r1, r2, r3};
  return __builtin_bit_cast(h8_t, v);
}

__device__ __forceinline__ f16_t mma(h8_t a, h8_t b, f16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Sixteen bytes per lane from sbase + voff to LDS at lds + 16 * lane.  Not known to the compiler's counting of
// loads: wait_loads() below is what makes the data valid.  The compiler learns from the output operand that m0 is written (m0
// is a reserved register: naming it a clobber has no effect); the s_nop is the wait state between that write and the load.
// (The base as an input that lives in m0 makes the compiler write it: the same work scheduled otherwise, 1 % slower on the
// shortest calls of owq_tile_few.)
__device__ __forceinline__ void load_to_lds(const void *sbase, u32 voff, u32 lds) {
  u32 m0;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" : "=&{m0}"(m0) : "s"(lds), "v"(voff), "s"(sbase) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ u32 lds_address(const void *p) {
  return (u32)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

__device__ __forceinline__ u32 pk_add(u32 a, u32 b) {
  return __builtin_bit_cast(u32, __builtin_bit_cast(h2_t, a) + __builtin_bit_cast(h2_t, b));
}
__device__ __forceinline__ u32 pk_sub(u32 a, u32 b) {
  return __builtin_bit_cast(u32, __builtin_bit_cast(h2_t, a) - __builtin_bit_cast(h2_t, b));
}
__device__ __forceinline__ u32 pk_dup(float v) {
  const u32 h = __builtin_bit_cast(unsigned short, (_Float16)v);
  return h | (h << 16);
}

// q - z of k-step S (0..7) of a block: the mask-and-OR operand plus nb[o] = -(2^(10-o) + z), exact.
template <int BITS, int S>
__device__ __forceinline__ h8_t a_exact(const u32 *wd, const Magic &M, const u32 *nb) {
  u32x4 v = __builtin_bit_cast(u32x4, a_operand<BITS, S>(wd, M));
  v.x = pk_add(v.x, nb[pair_offset(BITS, S, 0)]);
  v.y = pk_add(v.y, nb[pair_offset(BITS, S, 1)]);
  v.z = pk_add(v.z, nb[pair_offset(BITS, S, 2)]);
  v.w = pk_add(v.w, nb[pair_offset(BITS, S, 3)]);
  return __builtin_bit_cast(h8_t, v);
}

// Pair I of k-step S, masked, at the offset pair_offset() of its 16-bit window.
template <int BITS, int S, int I>
__device__ __forceinline__ u32 a_field(const u32 *wd) {
  if (BITS == 3) {
    constexpr int u = S >> 2, o = S & 3;
    const u32 d0 = wd[3 * u], d1 = wd[3 * u + 1], d2 = wd[3 * u + 2];
    if (o == 0) return I == 3 ? __builtin_amdgcn_perm(d1, d0, 0x06030401u) & field(3, 1) : d0 & field(3, 3 * I);
    if (o == 1) return I < 2 ? __builtin_amdgcn_perm(d1, d0, 0x06030401u) & field(3, 4 + 3 * I) : d1 & field(3, 2 + 3 * (I - 2));
    if (o == 2) return I == 3 ? d2 & field(3, 1) : __builtin_amdgcn_perm(d2, d1, 0x06030401u) & field(3, 3 * I);
    return (I < 2 ? d2 : d2 >> 6) & field(3, 4 + 3 * (I & 1));
  }
  return (I < 2 ? wd[S] : wd[S] >> 6) & field(4, I < 2 ? 4 * I : 2 + 4 * (I - 2));
}

// Pair I of (q - z) 2^-9 of k-step S (0..7) of a block, nz = -z 2^-9 in both halves, z an integer of at most 1024.  A masked
// pair read as fp16 is the subnormal q 2^(o-24), and one packed multiply-add by 2^(15-o) moves it and takes the zero point
// off, exactly.  As many instructions as mask-and-OR and an add, but one constant per row instead of one per offset.
template <int BITS, int S, int I>
__device__ __forceinline__ u32 a_small_pair(const u32 *wd, u32 nz) {
  constexpr int o = pair_offset(BITS, S, I);
  const _Float16 m = __builtin_bit_cast(_Float16, (unsigned short)((30 - o) << 10));      // 2^(15-o)
  return __builtin_bit_cast(u32, __builtin_elementwise_fma(__builtin_bit_cast(h2_t, a_field<BITS, S, I>(wd)), (h2_t){m, m},
                                                          __builtin_bit_cast(h2_t, nz)));
}
template <int BITS, int S>
__device__ __forceinline__ h8_t a_small(const u32 *wd, u32 nz) {
  return __builtin_bit_cast(h8_t, (u32x4){a_small_pair<BITS, S, 0>(wd, nz), a_small_pair<BITS, S, 1>(wd, nz),
                                          a_small_pair<BITS, S, 2>(wd, nz), a_small_pair<BITS, S, 3>(wd, nz)});
}

// Eight rows of y, or the `left` that there are, from LDS to any element of memory (rows of y need no alignment; an element at a
// time costs the kernels for prompts up to a third on layers whose rows are no multiple of eight).
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
__device__ __forceinline__ void store_rows(_Float16 *to, const _Float16 *from, int left) {
  if (left >= 8) {
    *reinterpret_cast<u32x4_any *>(to) = *reinterpret_cast<const u32x4 *>(from);
  } else {
    for (int q = 0; q < left; ++q) to[q] = from[q];
  }
}

}  // namespace owq
