// Batched path for more than 64 tokens (prompts, large decode batches) on the tile layout.
//
//     y[n,i] = sum_{j not weak} s_ig (q_ij - z_ig) x[n,j]  +  sum_t Ww_it x[n, idx_t]
//
// The passes of owq_tile.hip read the layer once per 64 tokens and spend half their time on launches, on
// partial results and on matrix instructions that one wave per SIMD cannot keep fed.  Here a workgroup of
// four waves owns 256 rows x 64 or 128 tokens and walks along the columns in blocks of 128; two workgroups share a compute
// unit and are not in step, so one's matrix instructions run under the other's vector instructions and waits:
//
//   x       goes from memory straight into LDS (16-byte direct loads, two buffers, asked for one block ahead), in rows
//           of 256 bytes whose 16-byte units are exchanged by the low bits of the token, so that operand reads are
//           free of bank conflicts; the weak columns of a block are then overwritten with zeros by the wave that
//           fetched them (the dense term must not see them, whatever they hold);
//   codes   go from registers into the operand (q - z) 2^-9, exactly (a_small); it is the B operand, so that a lane holds one
//           row of the result and sixteen tokens, and a row's step size is one register;
//   groups  the sums of a block start from zero and end on one multiply-add per value with the step size, in fp32, as many
//           roundings as blocks.  128 tokens of those sums and of the result would be all registers there are: the block is
//           worked through a token tile of 32 at a time, which keeps the weight operands (64 registers) instead of seven
//           eighths of the sums, and what follows from the lane is worked out where it is used;
//   weak    the fp16 weak columns are one more K range at the end, operands of both sides from LDS.
// Row groups with a zero point that is no integer of at most 1024 (found by the prep kernel) take what the rounded zero points
// lack off by a second set of matrix instructions with the constant operand rint(z) - z.
//
// One workgroup writes y itself when it owns all columns; when there are too few tiles for the chip the
// columns are cut into `split` ranges, fp32 partial results go to the scratch area and owq_wide_sum adds them
// in a fixed order.  No atomics: results are reproducible.
//
// What bounds it: power.  The card lowers its clock under matrix work on random data (4096 x 16384 at 2048 tokens, 3-bit,
// groups of 128: 304 us with 64-token tiles, 239 with x zero; a large fp16 library product of that size 224 and, on zeros,
// about 160), so every instruction beside the matrix work costs.  128 tokens per unpacked code instead of 64, in turn on one card:
// 298 -> 248 us there, 16384 x 4096 293 -> 273, 4-bit 5120 -> 13824 at 777 tokens 153 -> 145; vector instructions per matrix
// instruction 7.9 -> 5.4.  With a spill of two to five registers, which waits for the direct loads too, 275 becomes 304-324.
// (Sums kept in units of the block's step size and multiplied by ratios of step sizes instead: 251, 267 and 142, but a rounding
// per block on all of the sums, which does not leave a single column's weight exact beyond some 100 groups.)
// Where there are no two workgroups for a compute unit, one has eight waves, half the columns for four of them (HALVES): 16384 ->
// 4096 at 2048 tokens, 256 tiles, 281 -> 252 us (matrix pipe busy 43 % before); 13824 -> 5120, 4-bit, at 600 tokens 127 -> 110,
// at 2048 322 -> 279; 9000 -> 6016 at 1500 211 -> 178.  A barrier of four waves each, through counts in LDS, changed nothing.
// Row groups with rests take 422 instead of 446 us, 440 instead of 446, but 234 instead of 209: 378 workgroups are one round with
// twice the matrix work, 702 of 64 tokens were two shorter ones, and the plan does not know of the zero points.
#include <hip/hip_runtime.h>

#include "owq_internal.h"
#include "owq_tile_device.h"

namespace owq {
namespace {

constexpr int kWideRows = 256, kWideTokens = 64, kWideWaves = 4;
constexpr int kWideBufUnits = kWideTokens * 16;        // 16-byte units of one staged block: [token][16]
constexpr int kWideWeakUnits = 32 * 16;                // of 128 weak columns of a row tile
constexpr int kWideOutPitch = 264;                     // halves per token of the transposed result
// A workgroup's tile has NT / 2 times 64 tokens: two block buffers, later x at the weak columns and the weights.
constexpr int wide_lds(int NT) { return (NT == 2 ? 3 : 4) * kWideBufUnits * 16; }
static_assert(kWideBufUnits + kWideWaves * kWideWeakUnits <= 3 * kWideBufUnits, "a row tile's weak weights per wave beside x");
static_assert(2 * kWideBufUnits + kWideWaves * kWideWeakUnits <= 4 * kWideBufUnits, "the same beside x of 128 tokens");
static_assert(kWideTokens * kWideOutPitch * 2 <= wide_lds(2), "64 tokens of the result are transposed in the staging buffers");
constexpr int kWideSlotUnits = kWideWaves * 16 * 64;   // 16-byte units of a partial result (256 rows x 64 tokens, fp32)

constexpr int kFlagGroups = 16;          // groups of a row group that one workgroup of the prep kernel looks through

struct PrepArgs {
  const u32 *sz;
  const _Float16 *x;
  const int *weak_idx;
  int *flags;            // [n_rg][n_fl]
  _Float16 *xw;          // [ntok][xwpitch], zero beyond kp
  _Float16 *xcopy;       // [ntok][pitch], or nullptr
  int n_rg, n_fl, n_groups, d_out_pad, d_in, ntok, kp, xwpitch, pitch;
};

// The first n_rg x n_fl workgroups: does a row group hold a zero point that is no integer of at most 1024?  The
// others take four tokens each, a wave per token: the gather of x at the weak columns and, for rows that are no
// multiple of 16 bytes, a copy of x that is.  Latency is what it costs (a chain of two loads per element), so every
// wave has one token and independent loads (a grid-stride loop over all elements took 11.9 us on 2048 tokens).
__global__ __launch_bounds__(256) void owq_wide_prep(const PrepArgs a) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < a.n_rg * a.n_fl) {
    __shared__ int any;
    if (tid == 0) any = 0;
    __syncthreads();
    const int rg = blockIdx.x / a.n_fl, g0 = (blockIdx.x - rg * a.n_fl) * kFlagGroups;
    int row = rg * kWideRows + tid;
    if (row > a.d_out_pad - 1) row = a.d_out_pad - 1;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kFlagGroups; ++i) {
      int g = g0 + i;
      if (g > a.n_groups - 1) g = a.n_groups - 1;
      const float z = half_hi(a.sz[(size_t)g * a.d_out_pad + row]);
      bad |= !(__builtin_fabsf(z) <= 1024.f && z == __builtin_rintf(z));
    }
    if (bad) any = 1;
    __syncthreads();
    if (tid == 0) a.flags[blockIdx.x] = any;
    return;
  }
  const int n = ((int)blockIdx.x - a.n_rg * a.n_fl) * 4 + (tid >> 6), lane = tid & 63;
  if (n >= a.ntok) return;
  const _Float16 *xr = a.x + (size_t)n * a.d_in;
#pragma unroll 4
  for (int t = lane; t < a.xwpitch; t += 64) {
    const int j = a.weak_idx[t < a.kp ? t : 0];
    const _Float16 v = xr[j >= 0 ? j : 0];
    a.xw[(size_t)n * a.xwpitch + t] = (t < a.kp && j >= 0) ? v : (_Float16)0;
  }
  if (a.xcopy != nullptr) {
#pragma unroll 8
    for (int j = lane; j < a.pitch; j += 64) {
      const _Float16 v = xr[j < a.d_in ? j : 0];
      a.xcopy[(size_t)n * a.pitch + j] = j < a.d_in ? v : (_Float16)0;
    }
  }
}

struct WideArgs {
  const u32x4 *codes;
  const u32 *sz;               // [n_groups][d_out_pad]: fp16 scale | fp16 zero << 16
  const _Float16 *x;           // [ntok][pitch], 16-byte aligned rows
  const _Float16 *xw;          // [ntok][xwpitch]
  const u32x4 *weak_w;         // [d_out_pad][kunits]
  const unsigned char *wmask;  // bit e of byte i: column 8i+e is weak
  const int *flags;
  f4_t *slots;
  _Float16 *y;                 // [ntok][d_out]
  int pitch, xwpitch, d_in, d_out, d_out_pad, ntok;
  int nbp, nblk, n_rt, n_groups, bpg, kunits, n_rg, n_fl, n_tt;
  int full, split;             // the first `full` tiles have one workgroup each, the others `split` column ranges
};

// Tile `rem` of a launch: row group and tile of tokens (n_wt of them); four row groups x the token tiles are neighbours.
__device__ __forceinline__ void wide_tile(int rem, int n_rg, int n_wt, int &rg, int &tt) {
  const int g4 = rem / (4 * n_wt), gh = min(4, n_rg - 4 * g4), r2 = rem - g4 * 4 * n_wt;
  tt = r2 / gh;
  rg = 4 * g4 + (r2 - tt * gh);
}

template <int J> using Int = std::integral_constant<int, J>;
template <int N, int I = 0, class F>
__device__ __forceinline__ void each(F &&f) {
  if constexpr (I < N) {
    f(Int<I>{});
    each<N, I + 1>(f);
  }
}

// The weight operand of k-step S of a lane's row: (q - z) 2^-9, or q - z where rests of zero points are taken off too (2^-9
// of those may be none of fp16's numbers).
template <int BITS, bool REST, int S>
__device__ __forceinline__ h8_t wide_weights(const u32 *wd, u32 nz) {
  const h8_t v = a_small<BITS, S>(wd, nz);
  return REST ? v * (_Float16)512 : v;
}

// The columns [p0, p1) in blocks of 128 of the workgroup's tile: on return tot holds, per row tile and token tile of the
// wave, the scaled sums, a lane having one row (lane mod 32) and sixteen tokens.  `idle`: steps that the workgroup's other four
// waves have more.
template <int BITS, bool GROUPED, bool REST, int NT>
__device__ __forceinline__ void wide_columns(const WideArgs &a, unsigned char *lds, int rg, int n0, int p0, int p1, int idle, f16_t *tot) {
  constexpr int kBuf = NT * 512;                // 16-byte units of a buffer
  constexpr bool kRolled = GROUPED;             // one body for even and odd blocks, whose codes come late and into the same registers
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 3;
  const int b0 = 2 * p0, b1 = min(2 * p1, a.nblk);
  const u32 ldsb = lds_address(lds);

  // What follows from the lane is worked out anew where it is used (here()): kept, it does not fit the registers of 128 tokens.
  auto here = [&]() __attribute__((always_inline)) {
    u32 t = threadIdx.x;
    if (GROUPED && NT == 4) asm volatile("" : "+v"(t));
    return t & 63;
  };
  // ---- x: this wave fetches 8 NT tokens of the tile, four per load (a quarter wave per row); row n's units lie at ^ n.  (Sixteen
  // rows of 64 bytes per load and units in order would save the exclusive or per read: 4096 x 4096, 2048 tokens, 75 -> 82 us) ----
  const unsigned char *xtile = reinterpret_cast<const unsigned char *>(a.x) + (size_t)n0 * a.pitch * 2;
  const u32 pitch2 = (u32)(a.pitch * 2);
  const bool whole = n0 + 32 * NT <= a.ntok;
  auto fetch_x = [&](int b, int buf) __attribute__((always_inline)) {
    const unsigned char *src = xtile + (size_t)b * 256;
    const int left = a.d_in - b * 128;
    const u32 dst = ldsb + (u32)(buf * kBuf + w * 8 * NT * 16) * 16u, l = here();
    const u32 unit = (l & 15) ^ (l >> 4);       // of the first row; 4i rows on: ^ 4i
    if (whole && left >= 128) {
      const u32 xrow = (u32)(w * 8 * NT + (int)(l >> 4)) * pitch2;
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i)
        load_to_lds(src + (size_t)(4 * i) * pitch2, xrow + ((unit ^ (4 * i & 15)) << 4), dst + i * 1024u);
    } else {
      // tokens past the end: any row will do, their results are dropped; columns past the end of the row: unit 0 instead,
      // cleared below
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i) {
        const u32 n = (u32)min(w * 8 * NT + 4 * i + (int)(l >> 4), a.ntok - 1 - n0), oct = unit ^ (4 * i & 15);
        load_to_lds(src, n * pitch2 + ((int)oct * 8 < left ? oct << 4 : 0u), dst + i * 1024u);
      }
    }
  };
  // ---- codes and scales --------------------------------------------------------------------------------
  u32 cb[2][2][8];
  u32 szr[2], mkr[2];     // scale and zero point of a row; weak mask of 32 columns (a quarter wave each)
  const int rt0 = min(rg * 8 + 2 * w, a.n_rt - 1), rt1 = min(rg * 8 + 2 * w + 1, a.n_rt - 1), row0 = (rg * 8 + 2 * w) * 32;
  constexpr int CH = BITS == 3 ? 3 : 4;
  const unsigned char *tile0 = reinterpret_cast<const unsigned char *>(a.codes) + (size_t)(rt0 * a.nbp) * (CH * 1024);
  const unsigned char *tile1 = reinterpret_cast<const unsigned char *>(a.codes) + (size_t)(rt1 * a.nbp) * (CH * 1024);
  int fg = b0 / a.bpg, frem = b0 - fg * a.bpg;      // group of the block that is fetched
  typedef u32 u32x2 __attribute__((ext_vector_type(2)));
  // codes of block b (3-bit: one and a half of the three chunks of a pair of blocks) and the scales of its group
  auto fetch_codes = [&](int b, auto tag) __attribute__((always_inline)) {
    constexpr int R = decltype(tag)::value;
    const u32 l = here();
    u32 unit = l * 16u;         // (opaque: as a shift of the lane it becomes part of 64-bit address arithmetic)
    asm volatile("" : "+v"(unit));
    const bool odd = kRolled ? (b & 1) != 0 : R != 0;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const unsigned char *tile = (t ? tile1 : tile0) + (u32)(b >> 1) * (u32)(CH * 1024);
      u32 *dst = cb[R][t];
      if (BITS == 4) {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(tile + (odd ? 2048u : 0u) + unit);
        const u32x4 u = *reinterpret_cast<const u32x4 *>(tile + (odd ? 3072u : 1024u) + unit);
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
        dst[4] = u.x; dst[5] = u.y; dst[6] = u.z; dst[7] = u.w;
      } else {
        const u32 at[3] = {odd ? 1032u : 0u, odd ? 2048u : 8u, odd ? 2056u : 1024u};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const u32x2 v = *reinterpret_cast<const u32x2 *>(tile + at[c] + unit);
          dst[2 * c] = v.x;
          dst[2 * c + 1] = v.y;
        }
      }
    }
    if (GROUPED) szr[R] = (a.sz + (size_t)min(fg, a.n_groups - 1) * (u32)a.d_out_pad)[(u32)min(row0 + (int)l, a.d_out_pad - 1)];
    mkr[R] = (reinterpret_cast<const u32 *>(a.wmask) + min(b, a.nblk - 1) * 4)[l >> 4];
    const bool wrap = frem + 1 == a.bpg;
    fg += wrap ? 1 : 0;
    frem = wrap ? 0 : frem + 1;
  };

  u32 nz[2], nr[2];       // of the lane's two rows, in both halves: -z 2^-9, z rounded where it is no integer; what that lacks
  float sc[2];            // their step sizes
  auto take_sz = [&](u32 v) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const u32 u = (u32)__builtin_amdgcn_ds_bpermute((int)(t * 32 + (here() & 31)) * 4, (int)v);
      const float z = half_hi(u), z1 = REST ? __builtin_amdgcn_fmed3f(__builtin_rintf(z), -1024.f, 1024.f) : z;
      sc[t] = REST ? half_lo(u) : half_lo(u) * 0x1p9f;
      nz[t] = pk_dup(z1 * -0x1p-9f);
      if (REST) nr[t] = pk_dup(z1 - z);
    }
  };
  f16_t zero, part[GROUPED && REST ? 4 : 1];
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
  for (int i = 0; i < 2 * NT; ++i) tot[i] = zero;

  if (!GROUPED) take_sz(a.sz[min(row0 + (int)here(), a.d_out_pad - 1)]);
  fetch_x(b0, 0);
  fetch_codes(b0, Int<0>{});

  auto step = [&](int b, auto tag) __attribute__((always_inline)) {
    constexpr int J = decltype(tag)::value;     // registers, and where the loop is not rolled the buffer too, of the block
    const int buf = kRolled ? b & 1 : J;
    wait_loads<0>();            // this wave's part of block b is in LDS, its codes are in registers
    // (said here to the compiler, which does not count the direct loads: its own wait, wherever a register of these is used
    // first, would be behind the next block's direct loads and wait for them too)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < (BITS == 3 ? 6 : 8); ++c) asm volatile("" : "+v"(cb[J][t][c]));
    if (GROUPED) asm volatile("" : "+v"(szr[J]));
    asm volatile("" : "+v"(mkr[J]));
    const int left = a.d_in - b * 128;
    if (__ballot(mkr[J] != 0u) != 0ull || left < 128) {
      const int l = (int)here(), d = l >> 4;
      u32 m = mkr[J];
      const int lv = left - 32 * d;
      if (lv < 32) m |= lv <= 0 ? 0xffffffffu : 0xffffffffu << lv;
      while (m) {
        const int col = 32 * d + __builtin_ctz(m);
        m &= m - 1;
#pragma unroll
        for (int i = 0; i < NT / 2; ++i) {
          const int n = w * 8 * NT + 16 * i + (l & 15);
          _Float16 *row = reinterpret_cast<_Float16 *>(lds + (buf * kBuf + n * 16) * 16);
          row[(((col >> 3) ^ (n & 15)) << 3) + (col & 7)] = (_Float16)0;
        }
      }
    }
    __syncthreads();
    const u32 xl = here();
    // (the dynamic LDS is all there is and begins at 0, so that the exchange of units is one of address bits)
    u32 xsw = ldsb + (kRolled ? buf * kBuf * 16 : 0) + (xl & 31) * 256u + (((xl >> 5) ^ (xl & 15)) << 4);
    auto x_of = [&](int i, int S) __attribute__((always_inline)) {
      if (GROUPED && NT == 4) asm volatile("" : "+v"(xsw));
      const u32 at = (xsw ^ (u32)(S << 5)) + (u32)((kRolled ? 0 : buf * kBuf * 16) + i * 32 * 256);
      return *reinterpret_cast<const __attribute__((address_space(3))) h8_t *>(at);
    };
    const int next = min(b + 1, 2 * p1 - 1);
    if constexpr (GROUPED && !REST) {
      // A token tile at a time.  The block's weight operands are made with the first one and kept for the others; the next
      // block's codes are asked for when those begin to be used up (a tile earlier, or a k-step, does not fit the registers).
      // The second row tile is one k-step behind, so that the matrix instructions of one run under the multiply-adds of the
      // other (16384 x 4096, a workgroup per compute unit: 286 -> 275 us).  The empty blocks keep the compiler from moving a
      // chain of pure operations past the scheduling barriers, which costs its sums' registers.
      h8_t xp, x0 = x_of(0, 0), av[2][8];
      f16_t s0, s1;
      take_sz(szr[J]);
      fetch_x(min(b + 1, b1 - 1), buf ^ 1);
      each<8 * NT + 1>([&](auto step_q) __attribute__((always_inline)) {
        constexpr int q = decltype(step_q)::value, i = q >> 3, S = q & 7, ip = (q - 1) >> 3, Sp = (q - 1) & 7;
        h8_t x1;
        if constexpr (q + 1 < 8 * NT) x1 = x_of((q + 1) >> 3, (q + 1) & 7);
        if constexpr (i == NT - 1 && S == 1) fetch_codes(next, Int<0>{});
        if constexpr (q < 8) av[0][S] = wide_weights<BITS, false, S>(cb[J][0], nz[0]);
        if constexpr (q > 0 && q <= 8) av[1][Sp] = wide_weights<BITS, false, Sp>(cb[J][1], nz[1]);
        if constexpr (q > 0) {
          s1 = mma(xp, av[1][Sp], Sp == 0 ? zero : s1);
          asm volatile("" : "+v"(s1));
        }
        if constexpr (q > 0 && S == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) tot[ip][r] = __builtin_fmaf(s0[r], sc[0], tot[ip][r]);
          asm volatile("" : "+v"(tot[ip]));
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (q < 8 * NT) {
          s0 = mma(x0, av[0][S], S == 0 ? zero : s0);
          asm volatile("" : "+v"(s0));
        }
        if constexpr (q > 0 && S == 0) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int r = 0; r < 16; ++r) tot[NT + ip][r] = __builtin_fmaf(s1[r], sc[1], tot[NT + ip][r]);
          asm volatile("" : "+v"(tot[NT + ip]));
        }
        xp = x0;
        if constexpr (q + 1 < 8 * NT) x0 = x1;
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
      // KT token tiles at a time share a weight operand; without groups the sums go on from block to block.  With groups
      // (and rests) the operands are made again for the next tiles: kept beside two tiles' sums they do not fit.
      constexpr int KT = GROUPED ? 2 : NT;
      h8_t xv[KT], av[2];
#pragma unroll
      for (int i = 0; i < KT; ++i) xv[i] = x_of(i, 0);
      if (GROUPED) take_sz(szr[J]);
      fetch_x(min(b + 1, b1 - 1), buf ^ 1);
      if (!kRolled) fetch_codes(next, Int<(J ^ 1)>{});
#pragma unroll
      for (int t = 0; t < 2; ++t) av[t] = wide_weights<BITS, REST, 0>(cb[J][t], nz[t]);
      each<8 * (NT / KT)>([&](auto step_q) __attribute__((always_inline)) {
        constexpr int q = decltype(step_q)::value, i0 = (q >> 3) * KT, S = q & 7, qn = q + 1 < 8 * (NT / KT) ? q + 1 : q, Sn = qn & 7;
        h8_t xn[KT];
        if constexpr (qn > q) {
#pragma unroll
          for (int i = 0; i < KT; ++i) xn[i] = x_of((qn >> 3) * KT + i, Sn);
        }
        if constexpr (kRolled && qn == q) fetch_codes(next, Int<0>{});
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < KT; ++i) {
            f16_t &c = GROUPED ? part[t * KT + i] : tot[t * NT + i];
            c = mma(xv[i], av[t], GROUPED && S == 0 ? zero : c);
          }
        if (REST) {
          asm volatile("" : "+v"(nr[0]), "+v"(nr[1]));
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < KT; ++i) {
              f16_t &c = GROUPED ? part[t * KT + i] : tot[t * NT + i];
              c = mma(xv[i], __builtin_bit_cast(h8_t, (u32x4){nr[t], nr[t], nr[t], nr[t]}), c);
            }
        }
        if constexpr (qn > q) {
          // (or the compiler keeps the first token tiles' operands for the next ones)
          if constexpr (Sn == 0) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int c = 0; c < (BITS == 3 ? 6 : 8); ++c) asm volatile("" : "+v"(cb[J][t][c]));
          }
#pragma unroll
          for (int t = 0; t < 2; ++t) av[t] = wide_weights<BITS, REST, Sn>(cb[J][t], nz[t]);
#pragma unroll
          for (int i = 0; i < KT; ++i) xv[i] = xn[i];
        }
        if constexpr (GROUPED) {
#pragma unroll
          for (int i = 0; i < 2 * KT; ++i) asm volatile("" : "+v"(part[i]));
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (GROUPED && S == 7) {
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < KT; ++i) {
#pragma unroll
              for (int r = 0; r < 16; ++r)
                tot[t * NT + i0 + i][r] = __builtin_fmaf(part[t * KT + i][r], sc[t], tot[t * NT + i0 + i][r]);
              asm volatile("" : "+v"(tot[t * NT + i0 + i]));
            }
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    }
  };
  if constexpr (kRolled) {
    for (int b = b0; b < b1; ++b) step(b, Int<0>{});
  } else {
    int b = b0;
    while (b + 2 <= b1) {
      step(b, Int<0>{});
      step(b + 1, Int<1>{});
      b += 2;
    }
    if (b < b1) step(b, Int<0>{});
  }
  if (!GROUPED) {
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) tot[i][r] *= sc[i / NT];
  }
  for (int i = 0; i < idle; ++i) __syncthreads();
  wait_loads<0>();            // the loads past the end must not land in what the buffers are used for next
  __syncthreads();
}

// What follows the columns: the weak columns of the first column range, then y or a partial result.  NT token tiles from
// token n0 on, tot in the order of wide_columns; every wave of the workgroup is past its reads of the staging buffers.
// store = false: four waves whose tokens do not exist go the same way to the same barriers.
// slot: the partial result of the first 64 tokens, -1 where there is none; those of the next 64 are `split` further on.
template <int NT>
__device__ __forceinline__ void wide_finish(const WideArgs &a, unsigned char *lds, int rg, int n0, int s, int slot, bool store, f16_t *tot) {
  constexpr int kBuf = NT * 512;
  const int tid = threadIdx.x & 255, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), kg = lane >> 5;
  // ---- weak columns: 128 at a time, the gathered activations in the first buffer, each wave's weights (of one
  // row tile after the other) behind it ----
  if (s == 0) {
    const u32 ldsb = lds_address(lds), wofs = (u32)(kBuf + w * kWideWeakUnits) * 16u;
    for (int c = 0; 16 * c < a.kunits; ++c) {
      if (c > 0) __syncthreads();
      const unsigned char *xsrc = reinterpret_cast<const unsigned char *>(a.xw) + ((size_t)n0 * a.xwpitch + c * 128) * 2;
      const unsigned char *wsrc = reinterpret_cast<const unsigned char *>(a.weak_w) + (size_t)rg * kWideRows * a.kunits * 16 + c * 256;
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i) {
        const int n = w * 8 * NT + 4 * i + (lane >> 4);
        const int gn = min(n0 + n, a.ntok - 1) - n0;
        load_to_lds(xsrc, (u32)gn * (u32)(a.xwpitch * 2) + (u32)((lane & 15) ^ (n & 15)) * 16u, ldsb + (u32)((w * 8 * NT + 4 * i) * 16) * 16u);
      }
      const unsigned char *xb = lds + (lane & 31) * 256, *wb = lds + wofs + (lane & 31) * 256;
      const int ks = min(8, (a.kunits - 16 * c + 1) >> 1);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int r = 4 * i + (lane >> 4);
          const int gr = min(rg * kWideRows + w * 64 + t * 32 + r, a.d_out_pad - 1) - rg * kWideRows;
          int u = (lane & 15) ^ (r & 15);
          if (16 * c + u > a.kunits - 1) u = 0;
          load_to_lds(wsrc, (u32)gr * (u32)(a.kunits * 16) + (u32)u * 16u, ldsb + wofs + (u32)(4 * i * 16) * 16u);
        }
        wait_loads<0>();
        if (t == 0) __syncthreads();
        for (int S = 0; S < ks; ++S) {
          const int u = 2 * S + kg, off = (u ^ (lane & 15)) << 4;
          const u32x4 zero4 = {0u, 0u, 0u, 0u};
          const u32x4 wv = *reinterpret_cast<const u32x4 *>(wb + off);
          h8_t bv[NT];
#pragma unroll
          for (int i = 0; i < NT; ++i) bv[i] = *reinterpret_cast<const h8_t *>(xb + i * 32 * 256 + off);
          const h8_t av = __builtin_bit_cast(h8_t, 16 * c + u < a.kunits ? wv : zero4);
#pragma unroll
          for (int i = 0; i < NT; ++i) tot[NT * t + i] = mma(bv[i], av, tot[NT * t + i]);
        }
        // the next row tile's weights go where these were read from
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
    __syncthreads();
  }

  _Float16 *out = reinterpret_cast<_Float16 *>(lds);
#pragma unroll
  for (int half = 0; half < NT / 2; ++half, n0 += kWideTokens) {
    if (n0 >= a.ntok) break;
    if (slot >= 0) {
      if (!store) break;
      f4_t *dst = a.slots + ((size_t)slot + half * a.split) * kWideSlotUnits + (w * 16) * 64 + lane;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f16_t &v = tot[(i >> 1) * NT + 2 * half + (i & 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[(i * 4 + q) * 64] = (f4_t){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      }
      continue;
    }
    if (half > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f16_t &v = tot[(i >> 1) * NT + 2 * half + (i & 1)];
#pragma unroll
      for (int r = 0; r < 16; ++r)
        out[((i & 1) * 32 + 8 * (r >> 2) + 4 * kg + (r & 3)) * kWideOutPitch + w * 64 + (i >> 1) * 32 + (lane & 31)] = (_Float16)v[r];
    }
    __syncthreads();
    const int row0 = rg * kWideRows, ntok = store ? min(kWideTokens, a.ntok - n0) : 0;
    for (int e = tid; e < ntok * 32; e += 256) {
      const int n = e >> 5, r = (e & 31) * 8;
      store_rows(a.y + (size_t)(n0 + n) * a.d_out + row0 + r, out + n * kWideOutPitch + r, a.d_out - row0 - r);
    }
  }
}

// One workgroup = 256 rows x 32 NT tokens x one column range (a run of block pairs); a wave = 64 rows x 32 NT tokens.
// HALVES = 2: eight waves, the second four on the second half of the range, with buffers of their own.  The halves exchange
// the sums of 64 tokens each through LDS and finish 64 tokens each.
template <int BITS, bool GROUPED, int NT, int HALVES>
__global__ __launch_bounds__(256 * HALVES, 2) void owq_wide_mma(const WideArgs a) {
  static_assert(HALVES == 1 || NT == 4, "a half finishes 64 tokens");
  extern __shared__ u32x4 lds_units[];
  unsigned char *lds = reinterpret_cast<unsigned char *>(lds_units);
  // workgroups of one die (id mod 8) take neighbouring tiles, so that a die's L2 serves the codes and the activations to all of
  // them; the tiles with one workgroup come first
  const int n_wt = (a.n_tt + NT / 2 - 1) / (NT / 2), tiles = a.n_rg * n_wt;
  const int full = HALVES == 2 ? a.full : 0;
  const bool cut = HALVES == 1 || (int)blockIdx.x >= full;
  const int id = cut ? (int)blockIdx.x - full : (int)blockIdx.x, N = cut ? (int)gridDim.x - full : full, xcd = id & 7;
  const int lin = xcd * (N >> 3) + min(xcd, N & 7) + (id >> 3);
  const int s = cut ? lin / (tiles - full) : 0, rel = lin - s * (tiles - full);      // of its part
  int rg, tt;
  wide_tile(cut ? full + rel : rel, a.n_rg, n_wt, rg, tt);
  const int n0 = tt * 32 * NT, split = cut ? a.split : 1;
  // partial results lie by row group and tokens, or, if only some tiles have them, in the order of these
  const int slot = split > 1 ? (full == 0 ? rg * a.n_tt + tt * (NT / 2) : rel * (NT / 2)) * split + s : -1;
  const int p0 = s * a.nbp / split, p1 = (s + 1) * a.nbp / split;

  int rest = 0;
  for (int i = 0; i < a.n_fl; ++i) rest |= a.flags[rg * a.n_fl + i];
  f16_t tot[2 * NT];
  if constexpr (HALVES == 1) {
    if (rest != 0)
      wide_columns<BITS, GROUPED, true, NT>(a, lds, rg, n0, p0, p1, 0, tot);
    else
      wide_columns<BITS, GROUPED, false, NT>(a, lds, rg, n0, p0, p1, 0, tot);
    wide_finish<NT>(a, lds, rg, n0, s, slot, true, tot);
  } else {
    const int h = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), pm = (p0 + p1 + 1) >> 1;      // the first half is no shorter
    const int n_first = 2 * (pm - p0), n_second = min(2 * p1, a.nblk) - 2 * pm;
    unsigned char *own = lds + h * wide_lds(NT);
    if (rest != 0)
      wide_columns<BITS, GROUPED, true, NT>(a, own, rg, n0, h ? pm : p0, h ? p1 : pm, h ? n_first - n_second : 0, tot);
    else
      wide_columns<BITS, GROUPED, false, NT>(a, own, rg, n0, h ? pm : p0, h ? p1 : pm, h ? n_first - n_second : 0, tot);
    // token tiles 0 and 1 go to the first half, 2 and 3 to the second
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 3;
    f4_t *to = reinterpret_cast<f4_t *>(lds + (h ^ 1) * wide_lds(NT)) + w * 1024 + lane;
    const f4_t *from = reinterpret_cast<const f4_t *>(own) + w * 1024 + lane;
    f16_t mine[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f16_t &lo = tot[(i >> 1) * NT + (i & 1)], &hi = tot[(i >> 1) * NT + 2 + (i & 1)];
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[i][r] = h ? hi[r] : lo[r];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = h ? lo[4 * q + e] : hi[4 * q + e];
        to[(i * 4 + q) * 64] = v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4_t v = from[(i * 4 + q) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) mine[i][4 * q + e] += v[e];
      }
    __syncthreads();
    const bool store = n0 + 64 * h < a.ntok;
    wide_finish<2>(a, own, rg, store ? n0 + 64 * h : n0, s, slot < 0 ? -1 : slot + h * split, store, mine);
  }
}

// Adds the partial results of the tiles from `full` on in a fixed order: one workgroup per 64 rows x 64 tokens (what one wave of
// owq_wide_mma wrote), a wave per accumulator tile.  A tile of tokens has 64 << lg2.
__global__ __launch_bounds__(256) void owq_wide_sum(const f4_t *slots, _Float16 *y, int full, int n_rg, int n_tt, int lg2, int split, int ntok, int d_out) {
  __shared__ __align__(16) _Float16 out[64][72];
  const int tid = threadIdx.x, lane = tid & 63, i = tid >> 6;
  const int w = blockIdx.x & 3, rg = (blockIdx.x >> 2) / n_tt, tt = (blockIdx.x >> 2) - rg * n_tt;
  const int n0 = tt * kWideTokens, row0 = rg * kWideRows + w * 64;
  int tile = rg * n_tt + tt;
  if (full > 0) {             // its place in the order of wide_tile()
    const int rem = (rg & ~3) * ((n_tt + lg2) >> lg2) + (tt >> lg2) * min(4, n_rg - (rg & ~3)) + (rg & 3);
    if (rem < full) return;
    tile = ((rem - full) << lg2) + (tt & lg2);
  }
  if (n0 >= ntok || row0 >= d_out) return;
  const f4_t *src = slots + (size_t)tile * split * kWideSlotUnits + (w * 16 + i * 4) * 64 + lane;
  f4_t sum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) sum[q] = src[q * 64];
#pragma unroll 4
  for (int s = 1; s < split; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q] += src[(size_t)s * kWideSlotUnits + q * 64];
  const int n = (i & 1) * 32 + 4 * (lane >> 5), r = (i >> 1) * 32 + (lane & 31);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) out[n + 8 * q + e][r] = (_Float16)sum[q][e];
  __syncthreads();
  const int nn = min(64, ntok - n0);
  for (int e = tid; e < nn * 8; e += 256) {
    const int t = e >> 3, rr = (e & 7) * 8;
    store_rows(y + (size_t)(n0 + t) * d_out + row0 + rr, &out[t][rr], d_out - row0 - rr);
  }
}

typedef void (*wide_fn)(const WideArgs);
template <int NT, int HALVES>
wide_fn pick_wide_tokens(int bits, bool grouped) {
  if (bits == 3) return grouped ? owq_wide_mma<3, true, NT, HALVES> : owq_wide_mma<3, false, NT, HALVES>;
  return grouped ? owq_wide_mma<4, true, NT, HALVES> : owq_wide_mma<4, false, NT, HALVES>;
}
wide_fn pick_wide(int bits, bool grouped, int nt, int halves) {
  return nt != 4 ? pick_wide_tokens<2, 1>(bits, grouped) : halves == 2 ? pick_wide_tokens<4, 2>(bits, grouped) : pick_wide_tokens<4, 1>(bits, grouped);
}

// Kernel and work split of n_tt token tiles of 64 over n_rg row groups and nbp block pairs, with room for `slots` partial results;
// eight: workgroups of eight waves too.
struct WidePlan {
  int nt, halves, full, split;
  float us;
};
constexpr float kWide8 = 3.1f, kWide8Grouped = 3.6f;      // us per pair of blocks of a workgroup of eight waves, beside
constexpr float kWide8Us = 4.f, kWide8More = 9.f;         // the exchange of its halves; start and end of a round, which nothing runs under
constexpr int kWidePlans = 128;           // most token tiles that may go in two launches
constexpr float kWideLaunchUs = 14.f;     // start, first loads and end of a second launch
WidePlan wide_plan(bool grouped, int n_rg, int n_tt, int nbp, int64_t slots, bool eight) {
  WidePlan best{2, 1, 0, 1, 1e30f};
  if (n_tt == 0) return WidePlan{2, 1, 0, 1, 0.f};
  // us per pair of blocks: up to 128 workgroups, one and two on every compute unit, as costs to choose by.  30 whole calls (2048
  // to 16384 columns, 2048 to 13824 rows, 100 to 2048 tokens) took 0.94 to 1.19 of this and 14 us around it.  Row groups whose
  // zero points are no integers have twice the matrix work, which the host does not know of.
  constexpr float kPair[4][3] = {{1.65f, 1.85f, 3.7f}, {2.7f, 3.0f, 6.8f}, {2.13f, 2.3f, 4.2f}, {3.5f, 3.75f, 7.25f}};
  for (int nt = 2; nt <= 4; nt += 2) {
    const float *c = kPair[(grouped ? 2 : 0) + (nt == 4 ? 1 : 0)];
    const int tiles = n_rg * (nt == 4 ? (n_tt + 1) / 2 : n_tt);
    for (int s = 1; s <= 32 && s * 2 <= nbp + 1; ++s) {
      const int n = tiles * s, left = n % 512, pairs = (nbp + s - 1) / s;
      if (s > 1 && (int64_t)tiles * (nt / 2) * s > slots) break;
      const float last = left <= 128 ? c[0] : left <= 256 ? c[1] : c[1] + (c[2] - c[1]) * (0.53f + 0.47f * (left - 256) / 256);
      // rounds of 512 workgroups, which overlap at their ends, and for a split the launch of the sum
      const float us = pairs * (n / 512 * c[2] + (left ? last : 0.f)) - 2.2f * (n / 512 + (left ? 1 : 0) - 1) +
                       (s > 1 ? 1.6f + 0.009f * n_rg * n_tt * s : 0.f);
      if (us < best.us) best = WidePlan{nt, 1, 0, s, us};
    }
  }
  // Eight waves, one workgroup per compute unit: fewer than 512 tiles, of which 256, if there are as many, are a whole round and the
  // others are cut into column ranges that fill another.  (From 512 on two workgroups of four waves share a compute unit from
  // start to end and lose nothing: 5120 -> 13824, 4-bit, 1500 tokens, 648 tiles: 237 us, so 259.)
  // What is cut has to be better by a margin than one launch of tiles of 64 tokens, which the costs above are too high for: with
  // groups by what its workgroups' starts and ends take (14848 -> 8298, 4-bit, 903 tokens, 29 ranges: 263 us, so 248; 9600 -> 4752, 3-bit,
  // 1690 tokens, 19 ranges and two launches otherwise: 178, 197), with one scale per row by their share (3968 -> 7345, 4-bit, 1352
  // tokens 96, so 89).  With one scale per row two rounds of eight waves lose, too (10240 -> 10871, 3-bit, 1390 tokens 257, so 249).
  const float c8 = grouped ? kWide8Grouped : kWide8, four = best.us;
  float least = four;
  const bool small_tiles = best.nt == 2 && best.split == 1;
  const int tiles = n_rg * ((n_tt + 1) / 2), full = tiles / 256 * 256, rest = tiles - full, rounds = full / 256 + (rest ? 1 : 0);
  for (int s = 1; eight && tiles < 512 && s <= 32 && s * 2 <= nbp; ++s) {
    if (s > 1 && (rest == 0 || rest * s > 256 || (int64_t)rest * 2 * s > slots)) break;
    if (s == 1 && full > 0 && !grouped) continue;
    const int pairs = full / 256 * nbp + (rest ? (nbp + s - 1) / s : 0);
    const float us = kWide8Us + kWide8More * (rounds - 1) + c8 * pairs + (s > 1 ? 1.6f + 0.018f * rest * s : 0.f);
    const float margin = small_tiles && full > 0 && s > 1 ? (grouped ? 0.45f * s : 0.08f * four) : 0.f;
    if (us + margin < least) {
      least = us + margin;
      best = WidePlan{4, 2, s > 1 ? full : 0, s, us};
    }
  }
  return best;
}

}  // namespace

int prepare_tile_wide_kernels(const owq_layer_info_t &g, int32_t lds_limit) {
  if (2 * wide_lds(4) > lds_limit) return (int)hipErrorInvalidValue;
  int e = 0;
  for (int i = 0; i < 3 && e == 0; ++i) {
    const int nt = i == 0 ? 2 : 4, halves = i == 2 ? 2 : 1;
    e = (int)hipFuncSetAttribute(reinterpret_cast<const void *>(pick_wide(g.bits, g.n_groups > 1, nt, halves)),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds(nt) * halves);
  }
  return e;
}

int launch_tile_wide(const owq_layer_info_t &g, void *blob, void *scratch, uint64_t scratch_bytes, const void *x, void *y,
                     int32_t batch, void *stream) {
  uint8_t *base = static_cast<uint8_t *>(blob), *scr = static_cast<uint8_t *>(scratch);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int n_rg = (g.n_rt + 7) / 8, nblk = (g.d_in + kBlockCols - 1) / kBlockCols;
  const bool copy = (reinterpret_cast<uintptr_t>(x) & 15) != 0 || (g.d_in & 7) != 0;
  const int pitch = copy ? (g.d_in + 7) / 8 * 8 : g.d_in;
  const int xwpitch = (g.kp + 127) / 128 * 128;
  auto up = [](uint64_t n) { return (n + 255) / 256 * 256; };
  const int n_fl = (g.n_groups + kFlagGroups - 1) / kFlagGroups;
  const uint64_t flag_bytes = up((uint64_t)n_rg * n_fl * 4);
  const uint64_t tok_bytes = (uint64_t)xwpitch * 2 + (copy ? (uint64_t)pitch * 2 : 0);
  // tokens per pass: all of them, or what the scratch memory holds of the gathered (and copied) activations
  if (scratch_bytes < flag_bytes + 1024) return -1;
  int64_t cap = batch;
  if (tok_bytes) cap = (int64_t)((scratch_bytes - flag_bytes - 1024) / tok_bytes);
  if (cap < batch) cap = cap / kWideTokens * kWideTokens;
  if (cap < kWideTokens && cap < batch) return -1;
  const _Float16 *xp = static_cast<const _Float16 *>(x);
  _Float16 *yp = static_cast<_Float16 *>(y);

  for (int32_t t0 = 0; t0 < batch;) {
    const int left = batch - t0, pass = left < cap ? left : (int)cap, n_tt = (pass + kWideTokens - 1) / kWideTokens;
    const uint64_t xw_bytes = up((uint64_t)pass * xwpitch * 2), xc_bytes = copy ? up((uint64_t)pass * pitch * 2) : 0;
    PrepArgs pa;
    pa.sz = reinterpret_cast<const u32 *>(base + g.off_sz);
    pa.x = xp + (size_t)t0 * g.d_in;
    pa.weak_idx = reinterpret_cast<const int *>(base + g.off_weak_idx);
    pa.flags = reinterpret_cast<int *>(scr);
    pa.xw = reinterpret_cast<_Float16 *>(scr + flag_bytes);
    pa.xcopy = copy ? reinterpret_cast<_Float16 *>(scr + flag_bytes + xw_bytes) : nullptr;
    pa.n_rg = n_rg; pa.n_fl = n_fl; pa.n_groups = g.n_groups; pa.d_out_pad = g.d_out_pad; pa.d_in = g.d_in;
    pa.ntok = pass; pa.kp = g.kp; pa.xwpitch = xwpitch; pa.pitch = pitch;
    const int gather = xwpitch > 0 || copy ? (pass + 3) / 4 : 0;
    WideArgs wa;
    wa.codes = reinterpret_cast<const u32x4 *>(base + g.off_codes);
    wa.sz = pa.sz;
    wa.weak_w = reinterpret_cast<const u32x4 *>(base + g.off_weak_w);
    wa.wmask = base + g.off_wmask;
    wa.flags = pa.flags;
    const uint64_t used = flag_bytes + xw_bytes + xc_bytes;
    wa.slots = reinterpret_cast<f4_t *>(scr + used);
    const int64_t slots = scratch_bytes > used ? (int64_t)((scratch_bytes - used) / (kWideSlotUnits * 16)) : 0;
    wa.pitch = pitch; wa.xwpitch = xwpitch; wa.d_in = g.d_in; wa.d_out = g.d_out; wa.d_out_pad = g.d_out_pad;
    wa.nbp = g.nbp; wa.nblk = nblk; wa.n_rt = g.n_rt; wa.n_groups = g.n_groups;
    wa.bpg = g.group_size ? g.group_size / kBlockCols : g.nblk;
    wa.kunits = g.kp >> 3; wa.n_rg = n_rg; wa.n_fl = n_fl;
    // the token tiles in one or two launches: the first `a` of them and the rest, each with its own split
    int first = n_tt;
    const bool grouped = g.n_groups > 1;
    WidePlan whole = wide_plan(grouped, n_rg, n_tt, g.nbp, slots, true), some[kWidePlans];       // some[a]: of a token tiles
    float us = whole.us;
    // (one scale per row: a part of eight waves loses what the other part's launch costs, 11648 -> 7665, 3-bit, 1786 tokens 285 us, one
    // launch of four waves 268)
    for (int a = 1; a < n_tt && n_tt <= kWidePlans; ++a) some[a] = wide_plan(grouped, n_rg, a, g.nbp, slots, grouped);
    for (int a = 1; a < n_tt && n_tt <= kWidePlans; ++a) {
      const float v = some[a].us + some[n_tt - a].us + kWideLaunchUs;
      if (v < us) { us = v; first = a; }
    }
    hipLaunchKernelGGL(owq_wide_prep, dim3((unsigned)(n_rg * n_fl + gather)), dim3(256), 0, st, pa);
    for (int part = 0; part < 2; ++part) {
      const int ta = part ? first : 0, tb = part ? n_tt : first;
      if (ta >= tb) continue;
      const int p0 = ta * kWideTokens, p1 = tb * kWideTokens < pass ? tb * kWideTokens : pass;
      wa.n_tt = tb - ta;
      wa.ntok = p1 - p0;
      const WidePlan plan = first == n_tt ? whole : some[wa.n_tt];
      wa.full = plan.full;
      wa.split = plan.split;
      wa.x = copy ? pa.xcopy + (size_t)p0 * pitch : pa.x + (size_t)p0 * g.d_in;
      wa.xw = pa.xw + (size_t)p0 * xwpitch;
      wa.y = yp + (size_t)(t0 + p0) * g.d_out;
      const int nt2 = plan.nt / 2, n_wt = (wa.n_tt + nt2 - 1) / nt2, cut = n_rg * n_wt - plan.full;
      hipLaunchKernelGGL(pick_wide(g.bits, grouped, plan.nt, plan.halves), dim3((unsigned)(plan.full + cut * plan.split)),
                         dim3((unsigned)(256 * plan.halves)), wide_lds(plan.nt) * plan.halves, st, wa);
      if (wa.split > 1)
        hipLaunchKernelGGL(owq_wide_sum, dim3((unsigned)(n_rg * wa.n_tt * 4)), dim3(256), 0, st, (const f4_t *)wa.slots, wa.y, plan.full, n_rg,
                           wa.n_tt, nt2 - 1, wa.split, wa.ntok, g.d_out);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    t0 += pass;
  }
  return (int)hipSuccess;
}

}  // namespace owq
