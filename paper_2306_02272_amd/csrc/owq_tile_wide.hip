// Batched path for more than 64 tokens (prompts, large decode batches) on the tile layout.
//
//     y[n,i] = sum_{j not weak} s_ig (q_ij - z_ig) x[n,j]  +  sum_t Ww_it x[n, idx_t]
//
// The passes of owq_tile.hip read the layer once per 64 tokens and spend half their time on launches, on
// partial results and on matrix instructions that one wave per SIMD cannot keep fed.  Here a workgroup of
// four waves owns 256 rows x 64 tokens and walks along the columns in blocks of 128; two workgroups share a compute
// unit and are not in step, so one's matrix instructions run under the other's vector instructions and waits:
//
//   x       goes from memory straight into LDS (16-byte direct loads, two buffers, asked for one block ahead), in rows
//           of 256 bytes whose 16-byte units are exchanged by the low bits of the token, so that operand reads are
//           free of bank conflicts; the weak columns of a block are then overwritten with zeros by the wave that
//           fetched them (the dense term must not see them, whatever they hold);
//   codes   go from registers into the A operand: a pair is masked out of a dword and OR-ed into the
//           mantissas of 2^(10-o), then one packed add of -(2^(10-o) + z) leaves q - z, exactly: z is
//           rounded to an integer of at most 1024 first, and where a layer's zero points are no such
//           integers the rest r = z - rint(z) (exact in fp16) is taken off by a second set of matrix
//           instructions with the constant operand -r (a flag per row group, found by the prep kernel);
//   groups  every 128-column block starts its four accumulator tiles from zero and ends on one fused
//           multiply-add per value with the block's step size (in fp32); layers with one scale per row
//           scale once at the end;
//   weak    the fp16 weak columns are one more K range at the end, operands of both sides from LDS.
//
// One workgroup writes y itself when it owns all columns; when there are too few tiles for the chip the
// columns are cut into `split` ranges, fp32 partial results go to the scratch area and owq_wide_sum adds them
// in a fixed order.  No atomics: results are reproducible.
//
// What bounds it: beside its 32 matrix instructions a wave issues about 145 instructions of unpacking and 64 of scaling
// per block (by the counter 280 vector instructions in all).  4096 -> 16384 -> 4096, 3-bit, groups of 128, 2048 tokens: 2000 us in passes, 600-625 us here from box to box
// (915-880 TFLOP/s; a large fp16 library product reaches 1200 on the same card), the matrix cores busy 46 % of the cycles.
// On a box where this took 580, one workgroup of eight waves on 256 x 128 tokens per compute unit took 636, weak masks by a
// scalar load per block instead of with the codes 612.
#include <hip/hip_runtime.h>

#include "owq_internal.h"
#include "owq_tile_device.h"

namespace owq {
namespace {

constexpr int kWideRows = 256, kWideTokens = 64, kWideWaves = 4;
constexpr int kWideBufUnits = kWideTokens * 16;        // 16-byte units of one staged block: [token][16]
constexpr int kWideWeakUnits = 32 * 16;                // of 128 weak columns of a row tile
constexpr int kWideOutPitch = 264;                     // halves per token of the transposed result
constexpr int kWidePlanes = 3 * kWideBufUnits * 16;    // after the two block buffers (later: x at the weak columns and the weights)
constexpr int kWideLds = kWidePlanes + kWideWaves * 128 * 4;
static_assert(kWideBufUnits + kWideWaves * kWideWeakUnits <= 3 * kWideBufUnits, "a row tile's weak weights per wave beside x");
static_assert(kWideTokens * kWideOutPitch * 2 <= kWidePlanes, "the result is transposed in the staging buffers");
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
  int nbp, nblk, n_rt, n_groups, bpg, kunits, n_rg, n_fl, n_tt, split, yvec;
};

// The operands of one k-step: q - z of the wave's two row tiles, x of its two token tiles.
struct WideOps {
  h8_t a0, a1, b0, b1;
};
template <int BITS, int S>
__device__ __forceinline__ WideOps wide_ops(const u32 (*wd)[8], const unsigned char *xb, u32 xsw, const Magic &M, const u32 (*nb)[8]) {
  const unsigned char *p = xb + (xsw ^ (S << 5));
  WideOps o;
  o.b0 = *reinterpret_cast<const h8_t *>(p);
  o.b1 = *reinterpret_cast<const h8_t *>(p + 32 * 256);
  o.a0 = a_exact<BITS, S>(wd[0], M, nb[0]);
  o.a1 = a_exact<BITS, S>(wd[1], M, nb[1]);
  return o;
}

// K-steps S..7 of a block: the operands of step S + 1 are made while the matrix instructions of step S run.  The
// scheduling barriers keep the compiler from making all eight steps' operands first, which does not fit the registers.
// wd: the block's dwords of the wave's two row tiles; xb + xsw: the lane's token row, its units exchanged;
// acc 0,1 = row tile 0, token tiles 0,1; 2,3 = row tile 1.
template <int BITS, bool GROUPED, bool REST, int S>
struct WideSteps {
  static __device__ __forceinline__ void run(const WideOps &o, const u32 (*wd)[8], const unsigned char *xb, u32 xsw, const Magic &M,
                                             const u32 (*nb)[8], const u32 *nr, f16_t *acc, const f16_t &zero) {
    WideOps nx = o;
    if constexpr (S < 7) nx = wide_ops<BITS, (S < 7 ? S + 1 : 0)>(wd, xb, xsw, M, nb);
    constexpr bool kFirst = GROUPED && S == 0;
    acc[0] = mma(o.a0, o.b0, kFirst ? zero : acc[0]);
    acc[2] = mma(o.a1, o.b0, kFirst ? zero : acc[2]);
    acc[1] = mma(o.a0, o.b1, kFirst ? zero : acc[1]);
    acc[3] = mma(o.a1, o.b1, kFirst ? zero : acc[3]);
    if (REST) {
      const h8_t r0 = __builtin_bit_cast(h8_t, (u32x4){nr[0], nr[0], nr[0], nr[0]});
      const h8_t r1 = __builtin_bit_cast(h8_t, (u32x4){nr[1], nr[1], nr[1], nr[1]});
      acc[0] = mma(r0, o.b0, acc[0]);
      acc[1] = mma(r0, o.b1, acc[1]);
      acc[2] = mma(r1, o.b0, acc[2]);
      acc[3] = mma(r1, o.b1, acc[3]);
    }
    if (!REST) {
      // operand reads first, then a few vector instructions behind every matrix instruction
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    WideSteps<BITS, GROUPED, REST, S + 1>::run(nx, wd, xb, xsw, M, nb, nr, acc, zero);
  }
};
template <int BITS, bool GROUPED, bool REST>
struct WideSteps<BITS, GROUPED, REST, 8> {
  static __device__ __forceinline__ void run(const WideOps &, const u32 (*)[8], const unsigned char *, u32, const Magic &,
                                             const u32 (*)[8], const u32 *, f16_t *, const f16_t &) {}
};

template <int J> struct WideBuf {};
template <int J> __device__ std::integral_constant<int, J> wide_buf_index(WideBuf<J>);

// The columns [b0, b1) in blocks of 128 of the workgroup's tile: on return tot holds, per row tile and token
// tile of the wave, the scaled sums (grouped) or the raw ones.
template <int BITS, bool GROUPED, bool REST>
__device__ __forceinline__ void wide_columns(const WideArgs &a, unsigned char *lds, int rg, int n0, int p0, int p1, f16_t *tot) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 5, b0 = 2 * p0, b1 = min(2 * p1, a.nblk);
  const u32 ldsb = lds_address(lds);
  float *splane = reinterpret_cast<float *>(lds + kWidePlanes) + w * 128;
  u32 *zplane = reinterpret_cast<u32 *>(splane + 64);

  // ---- x: this wave fetches tokens 16w .. 16w+15 of the tile, four per load (a quarter wave per row) -----
  const int fn = w * 16 + (lane >> 4);          // + 4i
  u32 xoff[4];
  int xoct[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = fn + 4 * i;
    int gn = n0 + n;
    if (gn > a.ntok - 1) gn = a.ntok - 1;       // tokens past the end: any row will do, their results are dropped
    xoct[i] = (lane & 15) ^ (n & 15);
    xoff[i] = (u32)(gn - n0) * (u32)(a.pitch * 2) + (u32)xoct[i] * 16u;
  }
  const unsigned char *xtile = reinterpret_cast<const unsigned char *>(a.x) + (size_t)n0 * a.pitch * 2;
  auto fetch_x = [&](int b, int buf) __attribute__((always_inline)) {
    const unsigned char *src = xtile + (size_t)b * 256;
    const int left = a.d_in - b * 128;          // columns past the end of the row: unit 0 instead, cleared below
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32 off = xoct[i] * 8 < left ? xoff[i] : xoff[i] - (u32)xoct[i] * 16u;
      load_to_lds(src, off, ldsb + (u32)(buf * kWideBufUnits + (w * 16 + 4 * i) * 16) * 16u);
    }
  };
  // ---- codes and scales --------------------------------------------------------------------------------
  u32 cb[2][2][8];
  u32 szr[2], mkr[2];     // scale and zero point of a row; weak mask of 32 columns (a quarter wave each)
  const int rt0 = min(rg * 8 + 2 * w, a.n_rt - 1), rt1 = min(rg * 8 + 2 * w + 1, a.n_rt - 1);
  const int szrow = min((rg * 8 + 2 * w) * 32 + lane, a.d_out_pad - 1);
  constexpr int CH = BITS == 3 ? 3 : 4;
  const unsigned char *tile0 = reinterpret_cast<const unsigned char *>(a.codes) + (size_t)(rt0 * a.nbp) * (CH * 1024);
  const unsigned char *tile1 = reinterpret_cast<const unsigned char *>(a.codes) + (size_t)(rt1 * a.nbp) * (CH * 1024);
  const u32 *mask32 = reinterpret_cast<const u32 *>(a.wmask) + (lane >> 4);
  int fg = b0 / a.bpg, frem = b0 - fg * a.bpg;      // group of the block that is fetched
  typedef u32 u32x2 __attribute__((ext_vector_type(2)));
  // codes of block H of pair bp (3-bit: whole and half chunks) and the scales of its group
  auto fetch_codes = [&](int bp, auto tag) __attribute__((always_inline)) {
    constexpr int H = decltype(wide_buf_index(tag))::value;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const unsigned char *tile = (t ? tile1 : tile0) + (u32)bp * (u32)(CH * 1024) + lane * 16;
      u32 *dst = cb[H][t];
      const u32x4 v = *reinterpret_cast<const u32x4 *>(tile + (H ? 2048 : 0));
      if (BITS == 4) {
        const u32x4 u = *reinterpret_cast<const u32x4 *>(tile + (H ? 3072 : 1024));
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
        dst[4] = u.x; dst[5] = u.y; dst[6] = u.z; dst[7] = u.w;
      } else {
        const u32x2 u = *reinterpret_cast<const u32x2 *>(tile + 1024 + (H ? 8 : 0));
        if (H == 0) {
          dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w; dst[4] = u.x; dst[5] = u.y;
        } else {
          dst[0] = u.x; dst[1] = u.y; dst[2] = v.x; dst[3] = v.y; dst[4] = v.z; dst[5] = v.w;
        }
        dst[6] = dst[7] = 0u;
      }
    }
    // The mask last: the compiler does not count the direct loads, and its wait for the mask covers every load before it,
    // so that the scale, which is used behind the next block's direct loads, does not wait for those (5120 -> 13824 ->
    // 5120, 4-bit, 777 tokens: 312 -> 302 us; 4096 -> 16384 -> 4096, 3-bit, 2048 tokens: 605 -> 598)
    if (GROUPED) szr[H] = a.sz[(u32)min(fg, a.n_groups - 1) * (u32)a.d_out_pad + szrow];
    mkr[H] = mask32[min(2 * bp + H, a.nblk - 1) * 4];
    const bool wrap = frem + 1 == a.bpg;
    fg += wrap ? 1 : 0;
    frem = wrap ? 0 : frem + 1;
  };

  Magic M;
  M.init();
  u32 nb[2][8], nr[2];
  // scale and zero point of the wave's 64 rows (a lane each) to LDS; each lane takes the zero points of its
  // two rows back and makes the constants that turn the mask-and-OR operand into q - z
  auto take_sz = [&](u32 v) __attribute__((always_inline)) {
    const float z = half_hi(v);
    splane[lane] = half_lo(v);
    reinterpret_cast<float *>(zplane)[lane] = z;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float zt = reinterpret_cast<float *>(zplane)[t * 32 + (lane & 31)];
      const float z1 = __builtin_amdgcn_fmed3f(__builtin_rintf(zt), -1024.f, 1024.f);
      const u32 zz = pk_dup(-z1);
#pragma unroll
      for (int o = 0; o < 8; ++o) nb[t][o] = pk_sub(zz, M.m[o]);
      nr[t] = pk_dup(z1 - zt);
    }
  };
  f16_t acc[GROUPED ? 4 : 1], zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) tot[i] = zero;

  const u32 xsw = (u32)(lane & 31) * 256u + (u32)((kg ^ (lane & 15)) << 4);
  if (!GROUPED) take_sz(a.sz[szrow]);
  fetch_x(b0, 0);
  fetch_codes(p0, WideBuf<0>{});

  auto step = [&](int b, auto tag) __attribute__((always_inline)) {
    constexpr int J = decltype(wide_buf_index(tag))::value;
    wait_loads<0>();            // this wave's part of block b is in LDS, its codes are in registers
    const int left = a.d_in - b * 128;
    if (__ballot(mkr[J] != 0u) != 0ull || left < 128) {
      const int d = lane >> 4, n = w * 16 + (lane & 15);
      u32 m = mkr[J];
      const int lv = left - 32 * d;
      if (lv < 32) m |= lv <= 0 ? 0xffffffffu : 0xffffffffu << lv;
      _Float16 *row = reinterpret_cast<_Float16 *>(lds + (J * kWideBufUnits + n * 16) * 16);
      while (m) {
        const int col = 32 * d + __builtin_ctz(m);
        m &= m - 1;
        row[(((col >> 3) ^ (n & 15)) << 3) + (col & 7)] = (_Float16)0;
      }
    }
    __syncthreads();
    fetch_x(min(b + 1, b1 - 1), J ^ 1);
    fetch_codes(min((b + 1) >> 1, p1 - 1), WideBuf<(J ^ 1)>{});
    if (GROUPED) take_sz(szr[J]);
    const unsigned char *xb = lds + J * kWideBufUnits * 16;
    if constexpr (GROUPED) {
      __builtin_amdgcn_sched_barrier(0);
      WideSteps<BITS, true, REST, 0>::run(wide_ops<BITS, 0>(cb[J], xb, xsw, M, nb), cb[J], xb, xsw, M, nb, nr, acc, zero);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f4_t sc = *reinterpret_cast<const f4_t *>(splane + t * 32 + 8 * q + 4 * kg);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
              tot[t * 2 + nt][4 * q + e] = __builtin_fmaf(sc[e], acc[t * 2 + nt][4 * q + e], tot[t * 2 + nt][4 * q + e]);
        }
    } else {
      WideSteps<BITS, false, REST, 0>::run(wide_ops<BITS, 0>(cb[J], xb, xsw, M, nb), cb[J], xb, xsw, M, nb, nr, tot, zero);
    }
  };
  int b = b0;
  while (b + 2 <= b1) {
    step(b, WideBuf<0>{});
    step(b + 1, WideBuf<1>{});
    b += 2;
  }
  if (b < b1) step(b, WideBuf<0>{});
  if (!GROUPED) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4_t sc = *reinterpret_cast<const f4_t *>(splane + t * 32 + 8 * q + 4 * kg);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) tot[t * 2 + nt][4 * q + e] *= sc[e];
      }
  }
  wait_loads<0>();            // the loads past the end must not land in what the buffers are used for next
  __syncthreads();
}

// One workgroup = 256 rows x 64 tokens x one column range (a run of block pairs); a wave = 64 rows x 64 tokens.
template <int BITS, bool GROUPED>
__global__ __launch_bounds__(256, 2) void owq_wide_mma(const WideArgs a) {
  extern __shared__ u32x4 lds_units[];
  unsigned char *lds = reinterpret_cast<unsigned char *>(lds_units);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 5;
  // workgroups of one die (id mod 8) take neighbouring tiles: four row groups x the token tiles, so that a die's
  // L2 serves the codes and the activations to all of them
  const int N = gridDim.x, xcd = blockIdx.x & 7, lin = xcd * (N >> 3) + min(xcd, N & 7) + (int)(blockIdx.x >> 3);
  const int tiles = a.n_rg * a.n_tt, s = lin / tiles, rem = lin - s * tiles;
  const int g4 = rem / (4 * a.n_tt), gh = min(4, a.n_rg - 4 * g4), r2 = rem - g4 * 4 * a.n_tt;
  const int tt = r2 / gh, rg = 4 * g4 + (r2 - tt * gh);
  const int n0 = tt * kWideTokens;
  const int p0 = s * a.nbp / a.split, p1 = (s + 1) * a.nbp / a.split;

  f16_t tot[4];
  int rest = 0;
  for (int i = 0; i < a.n_fl; ++i) rest |= a.flags[rg * a.n_fl + i];
  if (rest != 0)
    wide_columns<BITS, GROUPED, true>(a, lds, rg, n0, p0, p1, tot);
  else
    wide_columns<BITS, GROUPED, false>(a, lds, rg, n0, p0, p1, tot);

  // ---- weak columns: 128 at a time, the gathered activations in the first buffer, each wave's weights (of one
  // row tile after the other) behind it ----
  if (s == 0) {
    const u32 ldsb = lds_address(lds), wofs = (u32)(kWideBufUnits + w * kWideWeakUnits) * 16u;
    for (int c = 0; 16 * c < a.kunits; ++c) {
      if (c > 0) __syncthreads();
      const unsigned char *xsrc = reinterpret_cast<const unsigned char *>(a.xw) + ((size_t)n0 * a.xwpitch + c * 128) * 2;
      const unsigned char *wsrc = reinterpret_cast<const unsigned char *>(a.weak_w) + (size_t)rg * kWideRows * a.kunits * 16 + c * 256;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = w * 16 + 4 * i + (lane >> 4);
        const int gn = min(n0 + n, a.ntok - 1) - n0;
        load_to_lds(xsrc, (u32)gn * (u32)(a.xwpitch * 2) + (u32)((lane & 15) ^ (n & 15)) * 16u, ldsb + (u32)((w * 16 + 4 * i) * 16) * 16u);
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
          const h8_t b0v = *reinterpret_cast<const h8_t *>(xb + off), b1v = *reinterpret_cast<const h8_t *>(xb + 32 * 256 + off);
          const h8_t av = __builtin_bit_cast(h8_t, 16 * c + u < a.kunits ? wv : zero4);
          tot[2 * t] = mma(av, b0v, tot[2 * t]);
          tot[2 * t + 1] = mma(av, b1v, tot[2 * t + 1]);
        }
        // the next row tile's weights go where these were read from
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
    __syncthreads();
  }

  if (a.split > 1) {
    f4_t *dst = a.slots + ((size_t)(rg * a.n_tt + tt) * a.split + s) * kWideSlotUnits + (w * 16) * 64 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        dst[(i * 4 + q) * 64] = (f4_t){tot[i][4 * q], tot[i][4 * q + 1], tot[i][4 * q + 2], tot[i][4 * q + 3]};
    return;
  }
  typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
  _Float16 *out = reinterpret_cast<_Float16 *>(lds);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const h4_t v = {(_Float16)tot[i][4 * q], (_Float16)tot[i][4 * q + 1], (_Float16)tot[i][4 * q + 2], (_Float16)tot[i][4 * q + 3]};
      *reinterpret_cast<h4_t *>(out + ((i & 1) * 32 + (lane & 31)) * kWideOutPitch + w * 64 + (i >> 1) * 32 + 8 * q + 4 * kg) = v;
    }
  __syncthreads();
  const int row0 = rg * kWideRows, ntok = min(kWideTokens, a.ntok - n0);
  if (a.yvec) {
    for (int e = tid; e < ntok * 32; e += 256) {
      const int n = e >> 5, r = (e & 31) * 8;
      if (row0 + r < a.d_out)
        *reinterpret_cast<u32x4 *>(a.y + (size_t)(n0 + n) * a.d_out + row0 + r) = *reinterpret_cast<const u32x4 *>(out + n * kWideOutPitch + r);
    }
  } else {
    for (int e = tid; e < ntok * 256; e += 256) {
      const int n = e >> 8, r = e & 255;
      if (row0 + r < a.d_out) a.y[(size_t)(n0 + n) * a.d_out + row0 + r] = out[n * kWideOutPitch + r];
    }
  }
}

// Adds the partial results of a tile in a fixed order: one workgroup per 64 rows x 64 tokens (what one wave of
// owq_wide_mma wrote), a wave per accumulator tile.
__global__ __launch_bounds__(256) void owq_wide_sum(const f4_t *slots, _Float16 *y, int n_tt, int split, int ntok, int d_out, int yvec) {
  __shared__ __align__(16) _Float16 out[64][72];
  const int tid = threadIdx.x, lane = tid & 63, i = tid >> 6;
  const int w = blockIdx.x & 3, tile = blockIdx.x >> 2, rg = tile / n_tt, tt = tile - rg * n_tt;
  const int n0 = tt * kWideTokens, row0 = rg * kWideRows + w * 64;
  if (n0 >= ntok || row0 >= d_out) return;
  const f4_t *src = slots + (size_t)tile * split * kWideSlotUnits + (w * 16 + i * 4) * 64 + lane;
  f4_t sum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) sum[q] = src[q * 64];
#pragma unroll 4
  for (int s = 1; s < split; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q] += src[(size_t)s * kWideSlotUnits + q * 64];
  const int n = (i & 1) * 32 + (lane & 31), r = (i >> 1) * 32 + 4 * (lane >> 5);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) out[n][r + 8 * q + e] = (_Float16)sum[q][e];
  __syncthreads();
  const int nn = min(64, ntok - n0);
  if (yvec) {
    for (int e = tid; e < nn * 8; e += 256) {
      const int t = e >> 3, rr = (e & 7) * 8;
      if (row0 + rr < d_out)
        *reinterpret_cast<u32x4 *>(y + (size_t)(n0 + t) * d_out + row0 + rr) = *reinterpret_cast<const u32x4 *>(&out[t][rr]);
    }
  } else {
    for (int e = tid; e < nn * 64; e += 256) {
      const int t = e >> 6, rr = e & 63;
      if (row0 + rr < d_out) y[(size_t)(n0 + t) * d_out + row0 + rr] = out[t][rr];
    }
  }
}

typedef void (*wide_fn)(const WideArgs);
wide_fn pick_wide(int bits, bool grouped) {
  if (bits == 3) return grouped ? owq_wide_mma<3, true> : owq_wide_mma<3, false>;
  return grouped ? owq_wide_mma<4, true> : owq_wide_mma<4, false>;
}

// Work split of `tiles` output tiles over nblk column blocks with room for `slots` partial results.
struct WidePlan {
  int split;
  float us;
};
WidePlan wide_plan(int tiles, int nbp, int64_t slots) {
  WidePlan best{1, 1e30f};
  if (tiles == 0) return WidePlan{1, 0.f};
  for (int s = 1; s <= 32 && s * 2 <= nbp + 1; ++s) {
    const int n = tiles * s, left = n % 512, pairs = (nbp + s - 1) / s;
    if (s > 1 && n > slots) break;
    // Two workgroups per compute unit: what a pair of blocks weighs with two of them (kPair2) and with one alone (kPair1),
    // against a split's launch of the sum and the traffic of a partial result.  These are not the times of this kernel
    // (4.8 us per pair: 4096 x 16384 at 2048 tokens, four rounds of 16 pairs in 310 us), so columns are split, and token tiles
    // divided, less often than those would have it.
    constexpr float kPair1 = 1.5f, kPair2 = 2.0f;
    const float us = (n / 512) * (pairs * kPair2 + 4.f) + (left == 0 ? 0.f : pairs * (left > 256 ? kPair2 : kPair1) + 4.f) +
                     (s > 1 ? 4.f + 0.03f * n : 0.f);
    if (us < best.us) best = WidePlan{s, us};
  }
  return best;
}

}  // namespace

int prepare_tile_wide_kernels(const owq_layer_info_t &g, int32_t lds_limit) {
  if (kWideLds > lds_limit) return (int)hipErrorInvalidValue;
  return (int)hipFuncSetAttribute(reinterpret_cast<const void *>(pick_wide(g.bits, g.n_groups > 1)),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kWideLds);
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
    hipLaunchKernelGGL(owq_wide_prep, dim3((unsigned)(n_rg * n_fl + gather)), dim3(256), 0, st, pa);

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
    wa.yvec = ((reinterpret_cast<uintptr_t>(y) & 15) == 0 && (g.d_out & 7) == 0) ? 1 : 0;
    // the token tiles in one or two launches: the first `a` of them and the rest, each with its own split
    int first = n_tt;
    float us = wide_plan(n_rg * n_tt, g.nbp, slots).us;
    for (int a = 1; a < n_tt; ++a) {
      const float v = wide_plan(n_rg * a, g.nbp, slots).us + wide_plan(n_rg * (n_tt - a), g.nbp, slots).us + 2.f;
      if (v < us) { us = v; first = a; }
    }
    for (int part = 0; part < 2; ++part) {
      const int ta = part ? first : 0, tb = part ? n_tt : first;
      if (ta >= tb) continue;
      const int p0 = ta * kWideTokens, p1 = tb * kWideTokens < pass ? tb * kWideTokens : pass;
      wa.n_tt = tb - ta;
      wa.ntok = p1 - p0;
      wa.split = wide_plan(n_rg * wa.n_tt, g.nbp, slots).split;
      wa.x = copy ? pa.xcopy + (size_t)p0 * pitch : pa.x + (size_t)p0 * g.d_in;
      wa.xw = pa.xw + (size_t)p0 * xwpitch;
      wa.y = yp + (size_t)(t0 + p0) * g.d_out;
      hipLaunchKernelGGL(pick_wide(g.bits, g.n_groups > 1), dim3((unsigned)(n_rg * wa.n_tt * wa.split)), dim3(256), kWideLds, st, wa);
      if (wa.split > 1)
        hipLaunchKernelGGL(owq_wide_sum, dim3((unsigned)(n_rg * wa.n_tt * 4)), dim3(256), 0, st, (const f4_t *)wa.slots, wa.y, wa.n_tt,
                           wa.split, wa.ntok, g.d_out, wa.yvec);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    t0 += pass;
  }
  return (int)hipSuccess;
}

}  // namespace owq
