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
//   codes   go from registers into the A operand (q - z) 2^-9, exactly (a_small);
//   groups  the accumulators hold the sums in units of the block's step size: before a block of another group they are
//           multiplied by (last step size / next), in fp32, and by the last one at the end.  With a second set of tiles that
//           takes the scaled blocks (as many vector instructions, 64 registers more) 128 tokens do not fit the registers.
//           What a ratio's rounding leaves goes into the next ratio, so all of them together are off by no more than one;
//           the rounding to y then takes the result as the multiplications leave it, good to 19 bits (settled);
//   weak    the fp16 weak columns are one more K range at the end, operands of both sides from LDS.
// Row groups with a zero point that is no integer of at most 1024 (groups: 240), or with a step size of zero or none that is finite, take
// wide_columns instead (found by the prep kernel): second set of tiles, rests of the zero points by a second set of matrix
// instructions with the constant operand rint(z) - z, 64 tokens at a time.
//
// One workgroup writes y itself when it owns all columns; when there are too few tiles for the chip the
// columns are cut into `split` ranges, fp32 partial results go to the scratch area and owq_wide_sum adds them
// in a fixed order.  No atomics: results are reproducible.
//
// What bounds it: power.  The card lowers its clock under matrix work on random data (4096 x 16384 at 2048 tokens, 3-bit,
// groups of 128: 304 us with 64-token tiles, 239 with x zero; a large fp16 library product of that size 224 and, on zeros,
// about 160), so every instruction beside the matrix work costs.  128 tokens per unpacked code instead of 64 take the
// vector instructions per matrix instruction from 7.9 to 4.7: 304 -> 248 us; 5120 -> 13824, 4-bit, 1500 tokens 270 -> 225.
// A schedule asked for with group barriers (five vector instructions behind every matrix instruction) 252, without 246.
#include <hip/hip_runtime.h>

#include "owq_internal.h"
#include "owq_tile_device.h"

namespace owq {
namespace {

constexpr int kWideRows = 256, kWideTokens = 64, kWideWaves = 4;
constexpr int kWideBufUnits = kWideTokens * 16;        // 16-byte units of one staged block: [token][16]
constexpr int kWideWeakUnits = 32 * 16;                // of 128 weak columns of a row tile
constexpr int kWideOutPitch = 264;                     // halves per token of the transposed result
// A workgroup's tile has NT / 2 times 64 tokens.  After the two block buffers (later: x at the weak columns and the weights):
// step sizes and zero points of a block, per wave.
constexpr int wide_planes(int NT) { return (NT == 2 ? 3 : 4) * kWideBufUnits * 16; }
constexpr int wide_lds(int NT) { return wide_planes(NT) + kWideWaves * 128 * 4; }
static_assert(kWideBufUnits + kWideWaves * kWideWeakUnits <= 3 * kWideBufUnits, "a row tile's weak weights per wave beside x");
static_assert(2 * kWideBufUnits + kWideWaves * kWideWeakUnits <= 4 * kWideBufUnits, "the same beside x of 128 tokens");
static_assert(kWideTokens * kWideOutPitch * 2 <= wide_planes(2), "64 tokens of the result are transposed in the staging buffers");
constexpr int kWideSlotUnits = kWideWaves * 16 * 64;   // 16-byte units of a partial result (256 rows x 64 tokens, fp32)

// |q - z| that wide_fast takes: what fp16 holds exactly; in groups, what is 19 bits times a step size (settled)
constexpr float kZeroLimit = 1024.f, kZeroLimitGroups = 240.f;

constexpr int kFlagGroups = 16;          // groups of a row group that one workgroup of the prep kernel looks through

struct PrepArgs {
  const u32 *sz;
  const _Float16 *x;
  const int *weak_idx;
  int *flags;            // [n_rg][n_fl]
  _Float16 *xw;          // [ntok][xwpitch], zero beyond kp
  _Float16 *xcopy;       // [ntok][pitch], or nullptr
  int n_rg, n_fl, n_groups, d_out, d_out_pad, d_in, ntok, kp, xwpitch, pitch;
  float zero_limit;      // largest zero point that wide_fast takes
};

// The first n_rg x n_fl workgroups: does a row group hold a zero point that is no integer of at most zero_limit, or a step
// size that is zero or no finite number?  The
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
    if (row > a.d_out - 1) row = a.d_out - 1;         // rows past the end have step size 0, and results that are dropped
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kFlagGroups; ++i) {
      int g = g0 + i;
      if (g > a.n_groups - 1) g = a.n_groups - 1;
      const u32 v = a.sz[(size_t)g * a.d_out_pad + row];
      const float z = half_hi(v), sc = __builtin_fabsf(half_lo(v));
      // (no short cuts: the compiler would wait for each load in a branch of its own)
      bad |= !((int)(__builtin_fabsf(z) <= a.zero_limit) & (int)(z == __builtin_rintf(z)) & (int)(sc > 0.f) & (int)(sc < INFINITY));
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
  int nbp, nblk, n_rt, n_groups, bpg, kunits, n_rg, n_fl, n_tt, split;
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

// The operands of one k-step of wide_fast: (q - z) 2^-9 of the wave's two row tiles, x of its NT token tiles.
template <int NT>
struct FastOps {
  h8_t a[2], b[NT];
};
template <int NT, int S>
__device__ __forceinline__ void fast_x(FastOps<NT> &o, const unsigned char *xb, u32 xsw) {
#pragma unroll
  for (int i = 0; i < NT; ++i) o.b[i] = *reinterpret_cast<const h8_t *>(xb + (xsw ^ (S << 5)) + i * 32 * 256);
}
template <int BITS, int NT, int S>
__device__ __forceinline__ void fast_codes(FastOps<NT> &o, const u32 (*wd)[8], const u32 *nz) {
#pragma unroll
  for (int t = 0; t < 2; ++t) o.a[t] = a_small<BITS, S>(wd[t], nz[t]);
}

// K-steps S..7 of a block: the operands of step S + 1 are made while the matrix instructions of step S run.  SCALE: the
// accumulators are brought to the step sizes of the block first (ratio: LDS, of the wave's 64 rows), a tile's share in front
// of its first matrix instruction.
template <int BITS, int NT, int S>
struct FastSteps {
  static __device__ __forceinline__ void run(const FastOps<NT> &o, const u32 (*wd)[8], const unsigned char *xb, u32 xsw, const u32 *nz,
                                             f16_t *acc) {
    FastOps<NT> nx = o;
    if constexpr (S < 7) {
      fast_x<NT, S + 1>(nx, xb, xsw);
      fast_codes<BITS, NT, S + 1>(nx, wd, nz);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[t * NT + i] = mma(o.a[t], o.b[i], acc[t * NT + i]);
    __builtin_amdgcn_sched_barrier(0);
    FastSteps<BITS, NT, S + 1>::run(nx, wd, xb, xsw, nz, acc);
  }
};
template <int BITS, int NT>
struct FastSteps<BITS, NT, 8> {
  static __device__ __forceinline__ void run(const FastOps<NT> &, const u32 (*)[8], const unsigned char *, u32, const u32 *, f16_t *) {}
};

// The columns [p0, p1) in blocks of 128 of the workgroup's tile, zero points integers of at most 1024 and step sizes finite
// and not zero: on return acc holds, per row tile and token tile of the wave, the scaled sums.
template <int BITS, bool GROUPED, int NT>
__device__ __forceinline__ void wide_fast(const WideArgs &a, unsigned char *lds, int rg, int n0, int p0, int p1, f16_t *acc) {
  constexpr int kBuf = NT * 512;                // 16-byte units of a buffer
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 5, b0 = 2 * p0, b1 = min(2 * p1, a.nblk);
  const u32 ldsb = lds_address(lds);
  float *splane = reinterpret_cast<float *>(lds + wide_planes(NT)) + w * 128, *zplane = splane + 64;

  // ---- x: this wave fetches 8 NT tokens of the tile, four per load (a quarter wave per row) -----
  const int fn = w * 8 * NT + (lane >> 4);      // + 4i
  u32 xoff[2 * NT];
#pragma unroll
  for (int i = 0; i < 2 * NT; ++i) {
    const int n = fn + 4 * i;
    int gn = n0 + n;
    if (gn > a.ntok - 1) gn = a.ntok - 1;       // tokens past the end: any row will do, their results are dropped
    xoff[i] = (u32)(gn - n0) * (u32)(a.pitch * 2) + (u32)(((lane & 15) ^ (n & 15)) * 16);
  }
  const unsigned char *xtile = reinterpret_cast<const unsigned char *>(a.x) + (size_t)n0 * a.pitch * 2;
  auto fetch_x = [&](int b, int buf) __attribute__((always_inline)) {
    const unsigned char *src = xtile + (size_t)b * 256;
    const int left = a.d_in - b * 128;          // columns past the end of the row: unit 0 instead, cleared below
    const u32 dst = ldsb + (u32)(buf * kBuf + w * 8 * NT * 16) * 16u;
    if (left >= 128) {
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i) load_to_lds(src, xoff[i], dst + i * 1024u);
    } else {
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i) {
        const int oct = (lane & 15) ^ ((fn + 4 * i) & 15);
        load_to_lds(src, oct * 8 < left ? xoff[i] : xoff[i] - (u32)oct * 16u, dst + i * 1024u);
      }
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
    if (GROUPED) szr[H] = a.sz[(u32)min(fg, a.n_groups - 1) * (u32)a.d_out_pad + szrow];
    mkr[H] = mask32[min(2 * bp + H, a.nblk - 1) * 4];
    const bool wrap = frem + 1 == a.bpg;
    fg += wrap ? 1 : 0;
    frem = wrap ? 0 : frem + 1;
  };

  u32 nz[2];              // -z 2^-9 of the lane's two rows
  float last;             // step size of the lane's row in the blocks so far: what the accumulators are in units of,
  float over = 0.f;       // and what the ratios' roundings have left of it
  float ratio = 1.f, was = 1.f;
  auto take_sz = [&](u32 v, bool first) __attribute__((always_inline)) {
    const float s = half_lo(v);
    if (GROUPED) {
      // (last + over) / s
      float rc = __builtin_amdgcn_rcpf(s);
      rc = __builtin_fmaf(__builtin_fmaf(-s, rc, 1.f), rc, rc);
      const float r = last * rc;
      ratio = first ? 1.f : __builtin_fmaf(__builtin_fmaf(-r, s, last) + over, rc, r);
      was = first ? s : last;
      splane[lane] = ratio;
    }
    last = s;
    zplane[lane] = half_hi(v) * -0x1p-9f;
#pragma unroll
    for (int t = 0; t < 2; ++t) nz[t] = pk_dup(zplane[t * 32 + (lane & 31)]);
  };
  // what the ratio's rounding leaves, in units of the new step size; not in front of the accumulators' multiplications, which wait
  // for the ratio (1 % of the whole there)
  auto carry = [&]() __attribute__((always_inline)) { over = (__builtin_fmaf(-ratio, last, was) + over) * __builtin_amdgcn_rcpf(ratio); };
#pragma unroll
  for (int i = 0; i < 2 * NT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  auto scale_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4_t sc = *reinterpret_cast<const f4_t *>(splane + t * 32 + 8 * q + 4 * kg);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < NT; ++i) acc[t * NT + i][4 * q + e] *= sc[e];
      }
  };

  const u32 xsw = (u32)(lane & 31) * 256u + (u32)((kg ^ (lane & 15)) << 4);
  last = 1.f;
  if (!GROUPED) take_sz(a.sz[szrow], true);
  fetch_x(b0, 0);
  fetch_codes(p0, WideBuf<0>{});

  auto step = [&](int b, auto tag) __attribute__((always_inline)) {
    constexpr int J = decltype(wide_buf_index(tag))::value;
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
      const int d = lane >> 4;
      u32 m = mkr[J];
      const int lv = left - 32 * d;
      if (lv < 32) m |= lv <= 0 ? 0xffffffffu : 0xffffffffu << lv;
      while (m) {
        const int col = 32 * d + __builtin_ctz(m);
        m &= m - 1;
#pragma unroll
        for (int i = 0; i < NT / 2; ++i) {
          const int n = w * 8 * NT + 16 * i + (lane & 15);
          _Float16 *row = reinterpret_cast<_Float16 *>(lds + (J * kBuf + n * 16) * 16);
          row[(((col >> 3) ^ (n & 15)) << 3) + (col & 7)] = (_Float16)0;
        }
      }
    }
    __syncthreads();
    // what the first k-step needs of LDS is asked for before the next block's loads go out
    const unsigned char *xb = lds + J * kBuf * 16;
    FastOps<NT> first;
    fast_x<NT, 0>(first, xb, xsw);
    if (GROUPED) take_sz(szr[J], b == b0);
    fetch_x(min(b + 1, b1 - 1), J ^ 1);
    fetch_codes(min((b + 1) >> 1, p1 - 1), WideBuf<(J ^ 1)>{});
    fast_codes<BITS, NT, 0>(first, cb[J], nz);
    if (GROUPED) {
      scale_acc();
      __builtin_amdgcn_sched_barrier(0);
      carry();
    }
    FastSteps<BITS, NT, 0>::run(first, cb[J], xb, xsw, nz, acc);
  };
  int b = b0;
  while (b + 2 <= b1) {
    step(b, WideBuf<0>{});
    step(b + 1, WideBuf<1>{});
    b += 2;
  }
  if (b < b1) step(b, WideBuf<0>{});
  splane[lane] = last * 0x1p9f;
  scale_acc();
  wait_loads<0>();            // the loads past the end must not land in what the buffers are used for next
  __syncthreads();
}

// The columns [b0, b1) in blocks of 128 of the workgroup's tile: on return tot holds, per row tile and token
// tile of the wave, the scaled sums (grouped) or the raw ones.
template <int BITS, bool GROUPED, bool REST, int PLANES>
__device__ __forceinline__ void wide_columns(const WideArgs &a, unsigned char *lds, int tid, int rg, int n0, int p0, int p1, f16_t *tot) {
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 5, b0 = 2 * p0, b1 = min(2 * p1, a.nblk);
  const u32 ldsb = lds_address(lds);
  float *splane = reinterpret_cast<float *>(lds + PLANES) + w * 128;
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

// A result of wide_fast in groups as the rounding to fp16 takes it: to 19 bits.  One column by itself gives s (q - z) x, 19 bits at
// most where x is a power of two, which often lies on a tie of fp16; the multiplications by the ratios leave some units of 2^-24
// there, which would break the tie either way.  To a sum that is not short it adds 2^-19 under fp16's own 2^-11.
__device__ __forceinline__ float settled(float v) {
  const u32 u = __builtin_bit_cast(u32, v), r = (u + 16u) & ~31u;
  return __builtin_bit_cast(float, (u & 0x7f800000u) == 0x7f800000u ? u : r);
}

// What follows the columns: the weak columns of the first column range, then y or a partial result.  NT token tiles from
// token n0 on, tot in the order of wide_fast; every wave of the workgroup is past its reads of the staging buffers.
// SETTLE: they come from ratios (settled).
template <int NT, bool SETTLE>
__device__ __forceinline__ void wide_finish(const WideArgs &a, unsigned char *lds, int tid, int rg, int n0, int s, f16_t *tot) {
  constexpr int kBuf = NT * 512;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), kg = lane >> 5;
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
          for (int i = 0; i < NT; ++i) tot[NT * t + i] = mma(av, bv[i], tot[NT * t + i]);
        }
        // the next row tile's weights go where these were read from
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
    __syncthreads();
  }

  typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
  _Float16 *out = reinterpret_cast<_Float16 *>(lds);
#pragma unroll
  for (int half = 0; half < NT / 2; ++half, n0 += kWideTokens) {
    if (n0 >= a.ntok) break;
    if (a.split > 1) {
      f4_t *dst = a.slots + ((size_t)(rg * a.n_tt + n0 / kWideTokens) * a.split + s) * kWideSlotUnits + (w * 16) * 64 + lane;
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
      for (int q = 0; q < 4; ++q) {
        h4_t hv;
#pragma unroll
        for (int e = 0; e < 4; ++e) hv[e] = (_Float16)(SETTLE ? settled(v[4 * q + e]) : v[4 * q + e]);
        *reinterpret_cast<h4_t *>(out + ((i & 1) * 32 + (lane & 31)) * kWideOutPitch + w * 64 + (i >> 1) * 32 + 8 * q + 4 * kg) = hv;
      }
    }
    __syncthreads();
    const int row0 = rg * kWideRows, ntok = min(kWideTokens, a.ntok - n0);
    for (int e = tid; e < ntok * 32; e += 256) {
      const int n = e >> 5, r = (e & 31) * 8;
      store_rows(a.y + (size_t)(n0 + n) * a.d_out + row0 + r, out + n * kWideOutPitch + r, a.d_out - row0 - r);
    }
  }
}

// One workgroup = 256 rows x 32 NT tokens x one column range (a run of block pairs); a wave = 64 rows x 32 NT tokens.
template <int BITS, bool GROUPED, int NT>
__global__ __launch_bounds__(256, 2) void owq_wide_mma(const WideArgs a) {
  extern __shared__ u32x4 lds_units[];
  unsigned char *lds = reinterpret_cast<unsigned char *>(lds_units);
  // workgroups of one die (id mod 8) take neighbouring tiles: four row groups x the token tiles, so that a die's
  // L2 serves the codes and the activations to all of them
  const int n_wt = (a.n_tt + NT / 2 - 1) / (NT / 2);
  const int N = gridDim.x, xcd = blockIdx.x & 7, lin = xcd * (N >> 3) + min(xcd, N & 7) + (int)(blockIdx.x >> 3);
  const int tiles = a.n_rg * n_wt, s = lin / tiles, rem = lin - s * tiles;
  const int g4 = rem / (4 * n_wt), gh = min(4, a.n_rg - 4 * g4), r2 = rem - g4 * 4 * n_wt;
  const int tt = r2 / gh, rg = 4 * g4 + (r2 - tt * gh);
  int n0 = tt * 32 * NT;
  const int p0 = s * a.nbp / a.split, p1 = (s + 1) * a.nbp / a.split;

  int general = 0;
  for (int i = 0; i < a.n_fl; ++i) general |= a.flags[rg * a.n_fl + i];
  if (general == 0) {
    f16_t acc[2 * NT];
    wide_fast<BITS, GROUPED, NT>(a, lds, rg, n0, p0, p1, acc);
    wide_finish<NT, GROUPED>(a, lds, (int)threadIdx.x, rg, n0, s, acc);
    return;
  }
  for (int half = 0; half < NT / 2 && n0 < a.ntok; ++half, n0 += kWideTokens) {
    f16_t tot[4];
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));           // what is made from it is made again for each half: kept over the loop it does not fit the registers
    if (half > 0) __syncthreads();          // the previous half's result has been read from where the next blocks go
    wide_columns<BITS, GROUPED, true, wide_planes(NT)>(a, lds, tid, rg, n0, p0, p1, tot);
    wide_finish<2, false>(a, lds, tid, rg, n0, s, tot);
  }
}

// Adds the partial results of a tile in a fixed order: one workgroup per 64 rows x 64 tokens (what one wave of
// owq_wide_mma wrote), a wave per accumulator tile.
// flags: those of owq_wide_prep where the accumulators were in units of step sizes, or nullptr.
__global__ __launch_bounds__(256) void owq_wide_sum(const f4_t *slots, _Float16 *y, const int *flags, int n_fl, int n_tt, int split, int ntok,
                                                    int d_out) {
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
  int general = flags == nullptr;
  for (int f = 0; f < n_fl && flags != nullptr; ++f) general |= flags[rg * n_fl + f];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) out[n][r + 8 * q + e] = (_Float16)(general ? sum[q][e] : settled(sum[q][e]));
  __syncthreads();
  const int nn = min(64, ntok - n0);
  for (int e = tid; e < nn * 8; e += 256) {
    const int t = e >> 3, rr = (e & 7) * 8;
    store_rows(y + (size_t)(n0 + t) * d_out + row0 + rr, &out[t][rr], d_out - row0 - rr);
  }
}

typedef void (*wide_fn)(const WideArgs);
template <int NT>
wide_fn pick_wide_tokens(int bits, bool grouped) {
  if (bits == 3) return grouped ? owq_wide_mma<3, true, NT> : owq_wide_mma<3, false, NT>;
  return grouped ? owq_wide_mma<4, true, NT> : owq_wide_mma<4, false, NT>;
}
wide_fn pick_wide(int bits, bool grouped, int nt) { return nt == 4 ? pick_wide_tokens<4>(bits, grouped) : pick_wide_tokens<2>(bits, grouped); }

// Kernel and work split of n_tt token tiles of 64 over n_rg row groups and nbp block pairs, with room for `slots` partial results.
struct WidePlan {
  int nt, split;
  float us;
};
constexpr float kWideLaunchUs = 14.f;     // start, first loads and end of a second launch
WidePlan wide_plan(bool grouped, int n_rg, int n_tt, int nbp, int64_t slots) {
  WidePlan best{2, 1, 1e30f};
  if (n_tt == 0) return WidePlan{2, 1, 0.f};
  // us per pair of blocks: up to 128 workgroups, one and two on every compute unit.  Fitted to 352 whole calls (2048 to 13824
  // columns, 2904 to 13824 rows, 160 to 1702 tokens, 1 to 6 ranges; 4.3 % root mean square).
  constexpr float kPair[4][3] = {{1.65f, 1.85f, 3.7f}, {2.7f, 3.0f, 6.8f}, {2.13f, 2.3f, 4.2f}, {3.5f, 3.75f, 7.25f}};
  for (int nt = 2; nt <= 4; nt += 2) {
    const float *c = kPair[(grouped ? 2 : 0) + (nt == 4 ? 1 : 0)];
    const int tiles = n_rg * (nt == 4 ? (n_tt + 1) / 2 : n_tt);
    for (int s = 1; s <= 32 && s * 2 <= nbp + 1; ++s) {
      const int n = tiles * s, left = n % 512, pairs = (nbp + s - 1) / s;
      if (s > 1 && (int64_t)n_rg * n_tt * s > slots) break;
      const float last = left <= 128 ? c[0] : left <= 256 ? c[1] : c[1] + (c[2] - c[1]) * (0.53f + 0.47f * (left - 256) / 256);
      // rounds of 512 workgroups, which overlap at their ends, and for a split the launch of the sum
      const float us = pairs * (n / 512 * c[2] + (left ? last : 0.f)) - 2.2f * (n / 512 + (left ? 1 : 0) - 1) +
                       (s > 1 ? 1.6f + 0.009f * n_rg * n_tt * s : 0.f);
      if (us < best.us) best = WidePlan{nt, s, us};
    }
  }
  return best;
}

}  // namespace

int prepare_tile_wide_kernels(const owq_layer_info_t &g, int32_t lds_limit) {
  if (wide_lds(4) > lds_limit) return (int)hipErrorInvalidValue;
  int e = 0;
  for (int nt = 2; nt <= 4 && e == 0; nt += 2)
    e = (int)hipFuncSetAttribute(reinterpret_cast<const void *>(pick_wide(g.bits, g.n_groups > 1, nt)),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds(nt));
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
    pa.n_rg = n_rg; pa.n_fl = n_fl; pa.n_groups = g.n_groups; pa.d_out = g.d_out; pa.d_out_pad = g.d_out_pad; pa.d_in = g.d_in;
    pa.ntok = pass; pa.kp = g.kp; pa.xwpitch = xwpitch; pa.pitch = pitch;
    pa.zero_limit = g.n_groups > 1 ? kZeroLimitGroups : kZeroLimit;
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
    float us = wide_plan(grouped, n_rg, n_tt, g.nbp, slots).us;
    for (int a = 1; a < n_tt && n_tt <= 128; ++a) {
      const float v = wide_plan(grouped, n_rg, a, g.nbp, slots).us + wide_plan(grouped, n_rg, n_tt - a, g.nbp, slots).us + kWideLaunchUs;
      if (v < us) { us = v; first = a; }
    }
    hipLaunchKernelGGL(owq_wide_prep, dim3((unsigned)(n_rg * n_fl + gather)), dim3(256), 0, st, pa);
    for (int part = 0; part < 2; ++part) {
      const int ta = part ? first : 0, tb = part ? n_tt : first;
      if (ta >= tb) continue;
      const int p0 = ta * kWideTokens, p1 = tb * kWideTokens < pass ? tb * kWideTokens : pass;
      wa.n_tt = tb - ta;
      wa.ntok = p1 - p0;
      const WidePlan plan = wide_plan(grouped, n_rg, wa.n_tt, g.nbp, slots);
      wa.split = plan.split;
      wa.x = copy ? pa.xcopy + (size_t)p0 * pitch : pa.x + (size_t)p0 * g.d_in;
      wa.xw = pa.xw + (size_t)p0 * xwpitch;
      wa.y = yp + (size_t)(t0 + p0) * g.d_out;
      const int n_wt = plan.nt == 4 ? (wa.n_tt + 1) / 2 : wa.n_tt;
      hipLaunchKernelGGL(pick_wide(g.bits, grouped, plan.nt), dim3((unsigned)(n_rg * n_wt * wa.split)), dim3(256),
                         wide_lds(plan.nt), st, wa);
      if (wa.split > 1)
        hipLaunchKernelGGL(owq_wide_sum, dim3((unsigned)(n_rg * wa.n_tt * 4)), dim3(256), 0, st, (const f4_t *)wa.slots, wa.y,
                           grouped ? pa.flags : (const int *)nullptr, n_fl, wa.n_tt, wa.split, wa.ntok, g.d_out);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    t0 += pass;
  }
  return (int)hipSuccess;
}

}  // namespace owq
