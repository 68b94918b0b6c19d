// Backward of the OWQ layer for weak-column tuning (paper, section "PEFT with Weak Column
// Tuning") on gfx950, from the packed tiles of the tile layout:
//
//     dx[n, j]           = sum_i dy[n, i] s[i, g(j)] (q[i, j] - z[i, g(j)])     j not weak
//     dx[n, weak_idx[t]] = sum_i dy[n, i] Ww[i, t]
//     dww[i, t]          = sum_n dy[n, i] x[n, weak_idx[t]]
//
// The dense part contracts over the rows i, while a lane of a packed tile holds eight
// consecutive COLUMNS of one row, which is what the forward product wants as a matrix-core
// operand and the wrong way round here.  The codes are therefore sent through the matrix core
// twice.  First as the A operand s (q - z), rounded to fp16 once, against a selection matrix (ones on a diagonal): the
// result is the same 32 x 32 block, but in the accumulator layout, where a lane holds one column and sixteen rows.
// Converted back to fp16 (exact) it is the B operand of the real product, whose A operand is dy, staged in operand
// order.  No LDS and no shuffles are needed for the turn.
//
// Per group of passes of 128 tokens (four, or up to sixteen of a small layer): staging (dy into operand order, on the first group also the weak
// columns and the activations at the weak columns); the small products (dww of the whole batch on the first group,
// dx at the weak columns in partial results); the product into fp32 partial results per range of rows, or, where there is
// one range, into dx; the sum of what partial results there are into fp16 dx.  A layer whose weak columns are more than an eighth of all takes a plain
// kernel for the weak columns of dx instead.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "owq_internal.h"
#include "owq_tile_device.h"

namespace owq {
namespace {

constexpr int kPassTokens = 128;     // tokens per pass: four accumulator tiles of 32 per wave
constexpr int kSplitMax = 16;        // most ranges of rows per block pair
constexpr int kWeakSplit = 32;       // ranges of rows of the product with the weak columns
constexpr int kLaunchPasses = 4;     // passes (of 128 tokens) that one set of launches takes, or
constexpr int kMorePasses = 16;      // up to so many where they do not fill the chip and their staged dy stays within
constexpr size_t kMoreBytes = 64u << 20;
// Fewer staging blocks of four token tiles than this do not fill the chip and take one tile each: 2048 -> 640 at 200 tokens, 22
// blocks, 4.4 -> 3.3 us; 4096 -> 4096 at 512, 260 blocks, 6.0 -> 5.6; but 7680 -> 10368 at 354, 489 blocks, 6.6 -> 8.0, and with rows
// of dy off the 8-byte grid 12032 -> 11155 at 65, 175 blocks, 5.1 -> 6.0.
constexpr int kStageBlocks = 320, kStageBlocksOff = 160;

// N 2-byte loads whose results get a use of their own after all of them have been issued, so
// that the compiler cannot move a load under the branch of a later select (loads under branches
// are waited for one by one).  Every address must be valid whatever the selects decide.
template <int N>
__device__ __forceinline__ void load_h(const _Float16 *const (&p)[N], _Float16 (&out)[N]) {
  u32 r[N];
#pragma unroll
  for (int e = 0; e < N; ++e) r[e] = __builtin_bit_cast(unsigned short, *p[e]);
#pragma unroll
  for (int e = 0; e < N; ++e) asm volatile("" : "+v"(r[e]));
#pragma unroll
  for (int e = 0; e < N; ++e) out[e] = __builtin_bit_cast(_Float16, (unsigned short)r[e]);
}

struct StageArgs {
  const _Float16 *dy;   // [batch][d_out]
  u32x4 *a_st;          // [pass][n_st][2][4 token tiles][64 lanes] units of 8 fp16
  int d_out, n_st, n0, batch, passes;      // n_st: row tiles staged per pass, the last one all zeros
};

// A unit: token 32 m + lane % 32 of the pass, rows 32 rt + 16 s + 4 h + {0..3} and
// the same + 8 (h = lane / 32): the order in which the turned codes hold their rows.  Block b of
// the staging takes two row tiles and NM tiles of 32 tokens of a pass (four, or one where there are few blocks), a thread
// one unit of each: the 64 rows x 2 bytes that its four waves read of a token are one 128-byte line, fetched by this
// block only.
template <int NM>
__device__ __forceinline__ void stage_dy(const StageArgs &a, unsigned b, int t) {
  const int pairs = (a.n_st + 1) >> 1;
  const int m0 = NM == 1 ? (int)(b & 3) : 0;
  if (NM == 1) b >>= 2;
  const int pr = (int)(b % (unsigned)pairs), pass = (int)(b / (unsigned)pairs);
  const int l = t & 63, s = (t >> 6) & 1, rt = 2 * pr + (t >> 7), h = l >> 5;
  if (pass >= a.passes || rt >= a.n_st) return;
  u32x4 *dst = a.a_st + (size_t)pass * a.n_st * 512 + ((size_t)rt * 2 + s) * 256 + m0 * 64 + l;
  const int n0 = a.n0 + kPassTokens * pass + 32 * m0 + (l & 31);
  h8_t v[NM];
  const int ia = 32 * rt + 16 * s + 4 * h;          // rows ia .. ia + 3 and ia + 8 .. ia + 11
  if (ia + 11 < a.d_out && (a.d_out & 3) == 0) {
    // both runs of four rows inside the matrix and 8-byte aligned (dy is 16-byte aligned)
    typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
    h4_t lo[NM], hi[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int n = n0 + 32 * m;
      const _Float16 *row = a.dy + (size_t)(n < a.batch ? n : a.batch - 1) * a.d_out + ia;
      lo[m] = *reinterpret_cast<const h4_t *>(row);
      hi[m] = *reinterpret_cast<const h4_t *>(row + 8);
    }
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = n0 + 32 * m < a.batch;
        v[m][e] = in ? lo[m][e] : (_Float16)0.f;
        v[m][4 + e] = in ? hi[m][e] : (_Float16)0.f;
      }
  } else {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int n = n0 + 32 * m;
      const _Float16 *p[8];
      _Float16 x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = ia + (e & 3) + 8 * (e >> 2);
        p[e] = a.dy + (size_t)(n < a.batch ? n : a.batch - 1) * a.d_out + (i < a.d_out ? i : a.d_out - 1);
      }
      load_h<8>(p, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = ia + (e & 3) + 8 * (e >> 2);
        v[m][e] = (n < a.batch && i < a.d_out) ? x[e] : (_Float16)0.f;
      }
    }
  }
#pragma unroll
  for (int m = 0; m < NM; ++m) dst[m * 64] = __builtin_bit_cast(u32x4, v[m]);
}

struct StageWeakArgs {
  const _Float16 *weak_w;   // [d_out_pad][kp]
  u32x4 *wst;               // [n_rt][2][kp32][64 lanes] units of 8 fp16
  int kp, kp32, n_rt;
};

// The weak columns in the same operand order: lane % 32 = weak column of the tile, rows as above.
__device__ __forceinline__ void stage_weak(const StageWeakArgs &a, long long u) {
  const long long total = (long long)a.n_rt * 2 * a.kp32 * 64;
  if (u >= total) return;
  const int l = (int)(u & 63);
  const long long q = u >> 6;
  const int tt = (int)(q % a.kp32), s = (int)((q / a.kp32) & 1), rt = (int)(q / a.kp32 / 2);
  const int t = 32 * tt + (l & 31), h = l >> 5;
  h8_t v;
  const _Float16 *p[8];
  _Float16 x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int i = 32 * rt + 16 * s + 4 * h + (e & 3) + 8 * (e >> 2);     // below d_out_pad; padded rows hold 0
    p[e] = a.weak_w + (size_t)i * a.kp + (t < a.kp ? t : a.kp - 1);
  }
  load_h<8>(p, x);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = t < a.kp ? x[e] : (_Float16)0.f;
  a.wst[u] = __builtin_bit_cast(u32x4, v);
}

struct ProdArgs {
  const u32 *codes;     // dwords of the packed tiles
  const u32 *sz;        // [G][d_out_pad] step size | zero point << 16
  const u32x4 *a_st;
  float *part;          // [pass][split][128][d_in_pad]
  _Float16 *dx;         // [ntok][d_in] instead, where one workgroup has all rows; or nullptr
  int d_in, ntok;
  int n_rt, nbp, chunks, d_out_pad, d_in_pad, blocks_per_group, n_groups, split, rt_per_split;
};

constexpr int kStepTiles = 4;                          // row tiles between two barriers
constexpr int kStepBytes = kStepTiles * 8192;          // staged dy of a step: 128 tokens x 128 rows
constexpr int kProdPlanes = 4 * kStepBytes;            // two buffers for either half of the rows; then per wave:
constexpr int kProdPlane = 2 * kStepTiles * 32 * 8;    // step sizes with zero points, and rests in operand order, of the rows of two steps
constexpr int kOutPitch = 72;                          // halves per token of 64 columns of the result
constexpr int kProdFlags = kProdPlanes + 8 * kProdPlane;        // per wave: it has met a large step size
constexpr int kProdLds = kProdFlags + 8 * 4;
constexpr float kLargeStep = 32.f;                     // times |q - z| of up to 1039 is what fp16 holds

template <int S> using KStep = std::integral_constant<int, S>;

// Eight values of a row times its step size.
__device__ __forceinline__ h8_t scaled(h8_t v, u32 ss) {
  const u32x4 u = __builtin_bit_cast(u32x4, v);
  auto mul = [&](u32 p) { return __builtin_bit_cast(u32, __builtin_bit_cast(h2_t, p) * __builtin_bit_cast(h2_t, ss)); };
  return __builtin_bit_cast(h8_t, (u32x4){mul(u.x), mul(u.y), mul(u.z), mul(u.w)});
}

// dx in partial results: a workgroup of eight waves takes 256 columns (a block pair) x 128 tokens x a range of row
// tiles; waves 0..3 take 64 columns each over the first half of the range, waves 4..7 the same columns over the second.
//
// What bounds it: per 32 rows x 64 columns x 128 tokens a wave issues 16 matrix instructions for the product and 4 for
// the turn: 1.05 PFLOP/s of both at 4096 -> 16384, 3-bit, 512 tokens, where a large fp16 library product on random data
// reaches 1.2 on the same card.  The step size leaves with the codes: s (q - z) is rounded to fp16 once, before the turn
// (relative error of 2^-11 at most, q - z being an integer; step sizes of 32 and above, whose products may be more than fp16
// holds, in a sweep of their own that other layers never enter), so dy is an operand as it is.  (It used to be
// multiplied by s in the loop, 32 instructions per row tile instead of 16, and needed a launch that finds its largest magnitude
// and a power of two against underflow.)  About 80 vector instructions per row tile, among the matrix instructions of the tile
// before: a turn in front of its own product leaves the matrix cores waiting for it, 86.5 against 82 us here, 183 against 173
// on 5120 -> 13824, 4-bit, 1000 tokens.  Operands of dy are read two reads ahead of their use.
// Staged dy comes in operand order by direct loads to LDS (no registers, no copies between register sets), step sizes
// and zero points lie in LDS by row; what a zero point lacks of an integer of at most 1024 is taken off by a side loop.
// A workgroup that has all rows of its columns stores dx itself, by way of LDS (fp32 partial results and their sum: 4096 rows
// of codes x 16384 columns, 512 tokens, 12.5 us for the sum, 5.1 now for the weak columns alone, the product 81.6 as before).
// Row tiles past the end of a range are left out one by one (whole steps with tiles of zeros: 11.1 instead of 8.6 us on
// 512 x 512, 24.0 instead of 20.0 on 2432 -> 2086 at 432 tokens).
template <int BITS>
__global__ __launch_bounds__(512, 2) void owq_bwd_product(const ProdArgs a) {
  extern __shared__ u32x4 lds_units[];
  unsigned char *lds = reinterpret_cast<unsigned char *>(lds_units);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), cw = w & 3, kh = w >> 2;
  int lane = threadIdx.x & 63, h = lane >> 5, n32 = lane & 31;
  // Workgroups go to the eight dies (each with its own L2) in turn.  The workgroups that read the
  // same rows of the staged dy (same pass, same range of rows, different block pairs) are given
  // ids that land on one die: die d takes a contiguous eighth of the (pass, range, block pair) order.
  const int N = gridDim.x, xcd = blockIdx.x & 7, id = xcd * (N >> 3) + min(xcd, N & 7) + (int)(blockIdx.x >> 3);
  const int bp = id % a.nbp, sp = (id / a.nbp) % a.split, pass = id / (a.nbp * a.split);
  const unsigned char *a_st = reinterpret_cast<const unsigned char *>(a.a_st) + (size_t)pass * (a.n_rt + 1) * 8192;
  const int lo = sp * a.rt_per_split, hi = min(lo + a.rt_per_split, a.n_rt), mid = lo + (hi - lo + 1) / 2;
  const int rt0 = kh ? mid : lo, rt1 = kh ? hi : mid;
  const int steps = (mid - lo + kStepTiles - 1) / kStepTiles;             // of either half (the first is not the shorter)
  const u32 ldsb = lds_address(lds);
  u32 *szplane = reinterpret_cast<u32 *>(lds + kProdPlanes + w * kProdPlane);             // [2][128]
  float *rplane = reinterpret_cast<float *>(szplane + 2 * kStepTiles * 32);               // [2][128]
  // this wave's 64 columns lie in one block (128 columns), hence in one group
  int g = (2 * bp + (cw >> 1)) / a.blocks_per_group;
  g = g < a.n_groups ? g : a.n_groups - 1;                          // columns past d_in: any group, they are not stored
  const u32 *sz = a.sz + (size_t)g * a.d_out_pad;
  // selection matrices: K-step t of the forward numbering holds columns 16 t .. 16 t + 15 of the
  // block; two of them side by side make a 32-column tile
  h8_t sel0, sel1;
  auto select = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sel0[e] = (n32 == 8 * h + e) ? (_Float16)1.f : (_Float16)0.f;
      sel1[e] = (n32 == 16 + 8 * h + e) ? (_Float16)1.f : (_Float16)0.f;
    }
  };
  select();
  f16_t acc[4][2], zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
  for (int m = 0; m < 4; ++m) acc[m][0] = acc[m][1] = zero;
  auto scale_acc = [&](float v) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[m][0][r] *= v;
        acc[m][1][r] *= v;
      }
  };
  float zacc[4] = {0.f, 0.f, 0.f, 0.f};
  u32 cd[kStepTiles][4];
  u32 szr[2];
  // codes of K-steps 4 cw .. 4 cw + 3 of the lane: 3 cw .. of its 12 or 4 cw .. of its 16 dwords.  Tiles past the range: the last
  // tile's (their dy is zero)
  auto fetch_codes = [&](int i, int rt) __attribute__((always_inline)) {
    const u32 *tile = a.codes + (size_t)(min(rt, a.n_rt - 1) * a.nbp + bp) * (u32)(a.chunks * 256);
    if (BITS == 4) {
      const u32x4 v = *reinterpret_cast<const u32x4 *>(tile + cw * 256 + lane * 4);
      cd[i][0] = v.x; cd[i][1] = v.y; cd[i][2] = v.z; cd[i][3] = v.w;
    } else {
#pragma unroll
      for (int v = 0; v < 3; ++v) cd[i][v] = tile[((3 * cw + v) >> 2) * 256 + lane * 4 + ((3 * cw + v) & 3)];
      cd[i][3] = 0u;
    }
  };
  auto fetch_sz = [&](int rt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) szr[i] = sz[min(32 * rt + 64 * i + lane, a.d_out_pad - 1)];
  };
  // the half's staged dy of a step: 8 KB per row tile, two of them by this wave
  auto fetch_dy = [&](int rt, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kStepTiles; ++i) {
      if (rt + i >= rt1) break;
      const unsigned char *src = a_st + (size_t)(rt + i) * 8192;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        load_to_lds(src, (u32)((2 * cw + j) * 1024 + lane * 16), ldsb + (u32)((2 * kh + buf) * kStepBytes + i * 8192 + (2 * cw + j) * 1024));
    }
  };
  // Step sizes with the zero points rounded; what those lack, times the step size, to where the lanes of either half of the
  // wave read eight of them at once: row 16 s + 8 b + 4 h + e of a row tile is element 4 b + e of unit (s, h).  True: some
  // zero point is no small integer.
  int any_large = 0;
  auto put_sz = [&](int buf, auto which) __attribute__((always_inline)) {
    constexpr bool large = decltype(which)::value;
    bool rest = false;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 64 * i + lane, q = r & 15;
      const int at = (r >> 4) * 16 + ((q >> 2) & 1) * 8 + (q >> 3) * 4 + (q & 3);
      const float z = half_hi(szr[i]), z1 = __builtin_amdgcn_fmed3f(__builtin_rintf(z), -1024.f, 1024.f);
      const float sc = half_lo(szr[i]);
      const bool l = __builtin_fabsf(sc) >= kLargeStep;
      const h2_t sz2 = {(_Float16)(l == large ? sc * (large ? 0x1p-2f : 0x1p9f) : 0.f), (_Float16)(z1 * -0x1p-9f)};
      any_large |= (int)(__ballot(l) != 0ull);
      szplane[buf * 128 + r] = __builtin_bit_cast(u32, sz2);
      rplane[buf * 128 + at] = sc * (z - z1);
      rest |= z != z1;
    }
    return !large && __ballot(rest) != 0ull;
  };
  // s (q - z) of a K-step of the forward numbering (16 columns) of the lane's row, rounded once; sz as put_sz left it
  auto weights = [&](int i, u32 szv, auto k_step) __attribute__((always_inline)) {
    constexpr int S = decltype(k_step)::value;
    return scaled(a_small<BITS, S>(cd[i], __builtin_amdgcn_perm(szv, szv, 0x03020302u)), __builtin_amdgcn_perm(szv, szv, 0x01000100u));
  };
  auto turned = [&](const f16_t &t, u32x4 *wb) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      u32 pk[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)       // fp16 numbers: exact whatever the rounding
        pk[e] = __builtin_bit_cast(u32, __builtin_amdgcn_cvt_pkrtz(t[8 * s + 2 * e], t[8 * s + 2 * e + 1]));
      wb[s] = (u32x4){pk[0], pk[1], pk[2], pk[3]};
    }
  };
  // Over all rows, with the step sizes below kLargeStep (large: with the others).
  auto sweep = [&](auto which) __attribute__((always_inline)) {
    u32x4 wb[2][2], wn[2][2];
    // ---- turn of the first row tile: s (q - z) from (row, eight columns) to (column, eight rows) per lane ----
    fetch_dy(rt0, 0);
    fetch_sz(rt0);
#pragma unroll
    for (int i = 0; i < kStepTiles; ++i) fetch_codes(i, rt0 + i);
    bool rest = put_sz(0, which);
    fetch_sz(rt0 + kStepTiles);
    {
      const u32 szv = szplane[n32];
      const f16_t t0 = mma(weights(0, szv, KStep<1>{}), sel1, mma(weights(0, szv, KStep<0>{}), sel0, zero));
      const f16_t t1 = mma(weights(0, szv, KStep<3>{}), sel1, mma(weights(0, szv, KStep<2>{}), sel0, zero));
      turned(t0, wb[0]);
      turned(t1, wb[1]);
    }
    fetch_codes(0, rt0 + kStepTiles);
    for (int st = 0; st < steps; ++st) {
      const int rt = rt0 + st * kStepTiles, nx = rt + kStepTiles, buf = st & 1;
      // The codes of the next step's first tile, asked for last, may be on their way.  (The compiler does not count the direct
      // loads: its own waits for the others would stand behind the next step's direct loads and wait for them too.)
      wait_loads<BITS == 3 ? 3 : 1>();
#pragma unroll
      for (int i = 1; i < kStepTiles; ++i)
#pragma unroll
        for (int v = 0; v < BITS; ++v) asm volatile("" : "+v"(cd[i][v]));
      asm volatile("" : "+v"(szr[0]), "+v"(szr[1]));
      __syncthreads();
      fetch_dy(nx, buf ^ 1);
      const bool rest_next = put_sz(buf ^ 1, which);
      fetch_sz(nx + kStepTiles);
      u32 szv[kStepTiles];                     // of the row tiles that are turned in this step: 1, 2, 3 and the next one's 0
#pragma unroll
      for (int i = 0; i < kStepTiles; ++i) szv[i] = szplane[(i + 1 < kStepTiles ? buf * 128 + 32 * (i + 1) : (buf ^ 1) * 128) + n32];
      const unsigned char *dyb = lds + (2 * kh + buf) * kStepBytes + lane * 16;
      if (rest) {                              // sum of dy s (z - rint z) per token
        const float *rp = rplane + buf * 128;
        for (int i = 0; i < 2 * min(kStepTiles, rt1 - rt); ++i) {
          const f4_t r0 = *reinterpret_cast<const f4_t *>(rp + (2 * i + h) * 8), r1 = *reinterpret_cast<const f4_t *>(rp + (2 * i + h) * 8 + 4);
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const h8_t d = *reinterpret_cast<const h8_t *>(dyb + (i * 4 + m) * 1024);
#pragma unroll
            for (int e = 0; e < 4; ++e) zacc[m] = __builtin_fmaf((float)d[4 + e], r1[e], __builtin_fmaf((float)d[e], r0[e], zacc[m]));
          }
        }
      }
      rest = rest_next;
      auto dy_of = [&](int i, int q) __attribute__((always_inline)) { return *reinterpret_cast<const h8_t *>(dyb + (i * 8 + q) * 1024); };
      // ---- product: dy against the turned weights of a row tile, and the turn of the next one (slot j) in between ----
#pragma unroll
      for (int i = 0; i < kStepTiles; ++i) {
        if (rt + i >= rt1) break;
        const int j = (i + 1) % kStepTiles;
        h8_t d0 = dy_of(i, 0), d1 = dy_of(i, 1), a0, a1;
        f16_t t;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int s = q >> 2, m = q & 3;
          const h8_t d2 = dy_of(i, q < 6 ? q + 2 : 7);
          acc[m][0] = mma(d0, __builtin_bit_cast(h8_t, wb[0][s]), acc[m][0]);
          acc[m][1] = mma(d0, __builtin_bit_cast(h8_t, wb[1][s]), acc[m][1]);
          if (q == 0) a0 = weights(j, szv[i], KStep<0>{});
          if (q == 1) a1 = weights(j, szv[i], KStep<1>{});
          if (q == 2) t = mma(a1, sel1, mma(a0, sel0, zero));
          if (q == 2) a0 = weights(j, szv[i], KStep<2>{});
          if (q == 3) a1 = weights(j, szv[i], KStep<3>{});
          if (q == 4) turned(t, wn[0]);
          if (q == 4) fetch_codes(j, nx + i + 1);
          if (q == 5) t = mma(a1, sel1, mma(a0, sel0, zero));
          if (q == 7) turned(t, wn[1]);
          d0 = d1;
          d1 = d2;
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          wb[0][s] = wn[0][s];
          wb[1][s] = wn[1][s];
        }
      }
    }
    wait_loads<0>();
  };
  sweep(std::false_type{});
  // Where the workgroup has met larger ones, whose products with q - z may be more than fp16 holds, another sweep takes
  // those, 2^-11 of them, and the sums are in that unit meanwhile (both exact).
  if (lane == 0) reinterpret_cast<int *>(lds + kProdFlags)[w] = any_large;
  __syncthreads();
  const u32x4 *f = reinterpret_cast<const u32x4 *>(lds + kProdFlags);
  const u32x4 f0 = f[0] | f[1];
  if (__builtin_amdgcn_readfirstlane((int)(f0.x | f0.y | f0.z | f0.w)) != 0) {
    scale_acc(0x1p-11f);
    asm volatile("" : "+v"(lane));     // what follows from the lane is worked out again: kept over both it does not fit the registers
    h = lane >> 5;
    n32 = lane & 31;
    select();
    sweep(std::true_type{});
    scale_acc(0x1p11f);
    __syncthreads();
  }
  // The rest of the zero points per token: both halves of the lanes, then from the operand layout (token = lane % 32)
  // to the accumulator layout (tokens along the registers); the planes of this wave have been read
  float *zbuf = reinterpret_cast<float *>(szplane);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const float z = zacc[m] + __shfl_xor(zacc[m], 32);
    if (h == 0) zbuf[m * 32 + n32] = z;
  }
  // second half of the rows to LDS, the first adds it and stores
  f4_t *xch = reinterpret_cast<f4_t *>(lds) + cw * 2048 + lane;
  if (kh == 1) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          xch[((m * 2 + c) * 4 + q) * 64] = (f4_t){acc[m][c][4 * q], acc[m][c][4 * q + 1], acc[m][c][4 * q + 2], acc[m][c][4 * q + 3]};
  }
  __syncthreads();
  if (kh == 1) return;
  const float *zother = reinterpret_cast<const float *>(lds + kProdPlanes + (w + 4) * kProdPlane);
  if (a.dx != nullptr) {
    // 32 tokens at a time through what has been read of the exchange, so that eight columns are stored at once
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f4_t o[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = xch[(m * 8 + q) * 64];
      _Float16 *out = reinterpret_cast<_Float16 *>(lds + cw * 32768 + m * 8192);
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int nl = 8 * (q & 3) + 4 * h + e;
          out[nl * kOutPitch + 32 * (q >> 2) + n32] =
              (_Float16)((acc[m][q >> 2][4 * (q & 3) + e] + o[q][e]) - (zbuf[32 * m + nl] + zother[32 * m + nl]));
        }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int nl = 8 * i + (lane >> 3), n = pass * kPassTokens + 32 * m + nl, j = 256 * bp + 64 * cw + 8 * (lane & 7);
        if (n < a.ntok) store_rows(a.dx + (size_t)n * a.d_in + j, out + nl * kOutPitch + 8 * (lane & 7), a.d_in - j);
      }
    }
    return;
  }
  float *part = a.part + ((size_t)pass * a.split + sp) * kPassTokens * a.d_in_pad;
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int j = 256 * bp + 64 * cw + 32 * c + n32;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4_t o = xch[((m * 2 + c) * 4 + q) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int nl = 32 * m + 8 * q + 4 * h + e;                // token of the pass that register 4 q + e holds
          part[(size_t)nl * a.d_in_pad + j] = (acc[m][c][4 * q + e] + o[e]) - (zbuf[nl] + zother[nl]);
        }
      }
    }
}

struct WeakProdArgs {
  const u32x4 *a_st;
  const u32x4 *wst;     // [n_rt][2][kp32][64 lanes]
  float *pw;            // [pass][wsplit][128][32 kp32]
  int n_rt, kp32, wsplit;
};

// dx at the weak columns in partial results: a workgroup takes a tile of 32 weak columns, 128 tokens and a range of row
// tiles, a wave 32 of the tokens.  A small product that is all latency: the loads of four row tiles go out together.
__device__ __forceinline__ void weak_product(const WeakProdArgs &a, int b) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5, n32 = lane & 31;
  const int tt = b % a.kp32, sp = (b / a.kp32) % a.wsplit, pass = b / (a.kp32 * a.wsplit);
  const int rt0 = (int)((long long)sp * a.n_rt / a.wsplit), rt1 = (int)((long long)(sp + 1) * a.n_rt / a.wsplit);
  const u32x4 *a_st = a.a_st + (size_t)pass * (a.n_rt + 1) * 512 + w * 64 + lane;
  const u32x4 *wst = a.wst + (size_t)tt * 64 + lane;
  f16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  constexpr int kTiles = 4;
  for (int rt = rt0; rt < rt1; rt += kTiles) {
    u32x4 d[kTiles][2], q[kTiles][2];
#pragma unroll
    for (int i = 0; i < kTiles; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        d[i][s] = a_st[(size_t)(rt + i < rt1 ? rt + i : a.n_rt) * 512 + s * 256];     // past the range: the tile of zeros
        q[i][s] = wst[(size_t)(2 * min(rt + i, a.n_rt - 1) + s) * a.kp32 * 64];
      }
#pragma unroll
    for (int i = 0; i < kTiles; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) acc = mma(__builtin_bit_cast(h8_t, d[i][s]), __builtin_bit_cast(h8_t, q[i][s]), acc);
  }
  float *pw = a.pw + ((size_t)pass * a.wsplit + sp) * kPassTokens * (32 * a.kp32);
#pragma unroll
  for (int r = 0; r < 16; ++r)
    pw[(size_t)(32 * w + 8 * (r >> 2) + 4 * h + (r & 3)) * (32 * a.kp32) + 32 * tt + n32] = acc[r];
}

struct SumArgs {
  const float *part;    // [pass][split][128][d_in_pad]
  const float *pw;      // [pass][wsplit][128][32 kp32], or nullptr
  const uint8_t *wmask; // bit j = column j is weak
  const int *weak_idx;
  _Float16 *dx;         // [batch][d_in]
  int d_in, d_in_pad, split, wsplit, n0, ntok, k, kp32, dense_blocks;
};

// dx: the partial results added in a fixed order.  Blocks below dense_blocks take 1024 columns
// each and skip the weak ones; the blocks after them take 256 weak columns each.
__global__ __launch_bounds__(256) void owq_bwd_sum(const SumArgs a) {
  if ((int)blockIdx.y >= a.ntok) return;
  const int pass = blockIdx.y / kPassTokens, nl = blockIdx.y % kPassTokens;
  const size_t base = (size_t)pass * a.split * kPassTokens;           // first (range, token) row of this pass
  if ((int)blockIdx.x < a.dense_blocks) {
    const int j = (blockIdx.x * 256 + threadIdx.x) * 4;            // four columns per thread (d_in_pad is a multiple of 256)
    if (j >= a.d_in) return;
    // four partial results in flight; past the last one it again, not added
    f4_t v = {0.f, 0.f, 0.f, 0.f};
    const float *src = a.part + (base + nl) * a.d_in_pad + j;
    for (int s = 0; s < a.split; s += 4) {
      f4_t r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = *reinterpret_cast<const f4_t *>(src + (size_t)min(s + i, a.split - 1) * kPassTokens * a.d_in_pad);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f4_t z = {0.f, 0.f, 0.f, 0.f};
        v += s + i < a.split ? r[i] : z;
      }
    }
    const u32 weak = (a.wmask[j >> 3] >> (j & 7)) & 15u;          // j is a multiple of 4: the four bits sit in one byte
    _Float16 *out = a.dx + (size_t)(a.n0 + blockIdx.y) * a.d_in + j;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (j + e < a.d_in && !((weak >> e) & 1u)) out[e] = (_Float16)v[e];
  } else {
    const int t = ((int)blockIdx.x - a.dense_blocks) * 256 + threadIdx.x;
    if (a.pw == nullptr || t >= a.k) return;
    const int col = a.weak_idx[t];
    if ((unsigned)col >= (unsigned)a.d_in) return;
    float v = 0.f;
    const size_t wbase = (size_t)pass * a.wsplit * kPassTokens;
#pragma unroll 8
    for (int s = 0; s < a.wsplit; ++s) v += a.pw[(wbase + (size_t)s * kPassTokens + nl) * (32 * a.kp32) + t];
    a.dx[(size_t)(a.n0 + blockIdx.y) * a.d_in + col] = (_Float16)v;
  }
}

struct WeakArgs {
  const _Float16 *dy;        // [batch][d_out]
  const _Float16 *weak_w;    // [d_out_pad][kp]
  const int *weak_idx;       // [kp], -1 = padding
  _Float16 *dx;
  int d_out, d_in, kp, n0, ntok;
};

// dx at the weak columns: 8 tokens x 8 weak columns per workgroup, rows dealt to the threads.
__global__ __launch_bounds__(256) void owq_bwd_weak(const WeakArgs a) {
  __shared__ float red[4][64];
  const int t0 = blockIdx.x * 8, nb = blockIdx.y * 8;
  float acc[8][8];
#pragma unroll
  for (int n = 0; n < 8; ++n)
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[n][t] = 0.f;
  for (int i = threadIdx.x; i < a.d_out; i += 256) {
    const h8_t wv = *reinterpret_cast<const h8_t *>(a.weak_w + (size_t)i * a.kp + t0);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int nl = nb + n < a.ntok ? nb + n : a.ntok - 1;         // past the end: the last token again, dropped below
      const float d = (float)a.dy[(size_t)(a.n0 + nl) * a.d_out + i];
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[n][t] = __builtin_fmaf(d, (float)wv[t], acc[n][t]);
    }
  }
  // sum over the 256 threads: inside the waves, then the four waves through LDS
  const int lane = threadIdx.x & 63, wv_id = threadIdx.x >> 6;
#pragma unroll
  for (int n = 0; n < 8; ++n)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float v = acc[n][t];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
      if (lane == 0) red[wv_id][n * 8 + t] = v;
    }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int n = threadIdx.x >> 3, t = threadIdx.x & 7;
    const float v = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
    const int col = a.weak_idx[t0 + t];
    if (nb + n < a.ntok && (unsigned)col < (unsigned)a.d_in) a.dx[(size_t)(a.n0 + nb + n) * a.d_in + col] = (_Float16)v;
  }
}

struct StageXArgs {
  const _Float16 *x;         // [batch][d_in]
  const int *weak_idx;
  u32x4 *xw_st;              // [token steps of 16][kp32][64 lanes] units of 8 fp16
  int d_in, k, kp32, batch, steps;
};

// The activations at the weak columns as A operands with the tokens on the contraction axis:
// lane % 32 = weak column of the tile, eight consecutive tokens per lane.
__device__ __forceinline__ void stage_x(const StageXArgs &a, long long u) {
  if (u >= (long long)a.steps * a.kp32 * 64) return;
  const int l = (int)(u & 63);
  const long long q = u >> 6;
  const int tt = (int)(q % a.kp32), ks = (int)(q / a.kp32);
  const int t = 32 * tt + (l & 31), h = l >> 5;
  int col = t < a.k ? a.weak_idx[t] : -1;
  if ((unsigned)col >= (unsigned)a.d_in) col = -1;
  h8_t v;
  const _Float16 *p[8];
  _Float16 xv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int n = 16 * ks + 8 * h + e;
    p[e] = a.x + (size_t)(n < a.batch ? n : a.batch - 1) * a.d_in + (col >= 0 ? col : 0);
  }
  load_h<8>(p, xv);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (col >= 0 && 16 * ks + 8 * h + e < a.batch) ? xv[e] : (_Float16)0.f;
  a.xw_st[u] = __builtin_bit_cast(u32x4, v);
}

struct StageAllArgs {
  StageArgs dy;
  StageWeakArgs weak;
  StageXArgs x;
  unsigned dy_blocks, weak_blocks;   // blocks [0, dy_blocks) stage dy, the next weak_blocks the weak columns, the rest x
  int narrow;                        // a block of dy takes one tile of 32 tokens instead of four
};

// All staging of a call in one launch: the three parts are independent of each other.
__global__ __launch_bounds__(256) void owq_bwd_stage_all(const StageAllArgs a) {
  const unsigned b = blockIdx.x;
  if (b < a.dy_blocks && a.narrow) stage_dy<1>(a.dy, b, (int)threadIdx.x);
  else if (b < a.dy_blocks) stage_dy<4>(a.dy, b, (int)threadIdx.x);
  else if (b < a.dy_blocks + a.weak_blocks) stage_weak(a.weak, (long long)(b - a.dy_blocks) * 256 + threadIdx.x);
  else stage_x(a.x, (long long)(b - a.dy_blocks - a.weak_blocks) * 256 + threadIdx.x);
}

struct DwwArgs {
  const _Float16 *dy;        // [batch][d_out]
  const u32x4 *xw_st;
  float *dww;                // [d_out][k]
  int d_out, k, kp32, batch, steps;
};

// dww[i, t] = sum_n x[n, idx[t]] dy[n, i] on the matrix cores: a workgroup owns 32 rows i and NTT
// tiles of 32 weak columns; its four waves deal the token steps among them and add their results
// through LDS in a fixed order.  The work is tiny and all latency: a wave sends out the loads of
// eight of its token steps at once.
template <int NTT>
__device__ __forceinline__ void dww_product(const DwwArgs &a, int bx, int by) {
  __shared__ float red[4][16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5;
  const int i = bx * 32 + (lane & 31), tt0 = by * NTT;
  const int ntt = a.kp32 - tt0 < NTT ? a.kp32 - tt0 : NTT;
  const int ic = i < a.d_out ? i : a.d_out - 1;
  f16_t acc[NTT];
#pragma unroll
  for (int c = 0; c < NTT; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
  constexpr int kSteps = 8;                          // token steps of a wave in flight together
  for (int ks = w; ks < a.steps; ks += 4 * kSteps) {
    h8_t b[kSteps];
    u32x4 xa[kSteps][NTT];
    const _Float16 *p[8 * kSteps];
    _Float16 v[8 * kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const int k2 = ks + 4 * u;                     // k2 >= steps: tokens past the batch, zeros
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int n = 16 * k2 + 8 * h + e;
        p[8 * u + e] = a.dy + (size_t)(n < a.batch ? n : a.batch - 1) * a.d_out + ic;
      }
      const int kc = k2 < a.steps ? k2 : a.steps - 1;
#pragma unroll
      for (int c = 0; c < NTT; ++c) xa[u][c] = a.xw_st[((size_t)kc * a.kp32 + (c < ntt ? tt0 + c : tt0)) * 64 + lane];
    }
    load_h<8 * kSteps>(p, v);
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        b[u][e] = (16 * (ks + 4 * u) + 8 * h + e < a.batch && i < a.d_out) ? v[8 * u + e] : (_Float16)0.f;
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int c = 0; c < NTT; ++c) acc[c] = mma(__builtin_bit_cast(h8_t, xa[u][c]), b[u], acc[c]);
  }
#pragma unroll
  for (int c = 0; c < NTT; ++c) {
    __syncthreads();                                 // every thread, every round: the trip count is fixed
#pragma unroll
    for (int r = 0; r < 16; ++r) red[w][r][lane] = acc[c][r];
    __syncthreads();
    if (c < ntt) {
      // this thread's share of the 16 x 64 results: registers 4 w .. 4 w + 3 = four consecutive weak columns
      f4_t v;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 4 * w + q;
        v[q] = (red[0][r][lane] + red[1][r][lane]) + (red[2][r][lane] + red[3][r][lane]);
      }
      const int t = 32 * (tt0 + c) + 8 * w + 4 * h;
      if (i < a.d_out) {
        float *out = a.dww + (size_t)i * a.k + t;
        if ((a.k & 3) == 0 && t + 3 < a.k) {
          *reinterpret_cast<f4_t *>(out) = v;        // 16-byte aligned: dww is, and k is a multiple of 4
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (t + q < a.k) out[q] = v[q];
        }
      }
    }
  }
}

// The two small products of a call in one launch: dww in the first blocks of the grid, dx at the weak columns in the
// others (either may be absent).
// Both move as many bytes as they wait: blocks that read the same lines (neighbouring row tiles of dy, the weak tiles of a range)
// land on one die, whose L2 then serves them.  5120 -> 13824, 1000 tokens: 22.2 -> 18.8 us, 4096 -> 16384, 512 tokens 11.9 -> 10.8.
template <int NTT>
__global__ __launch_bounds__(256) void owq_bwd_small(const DwwArgs da, const WeakProdArgs wa, int dww_rows, int dww_blocks) {
  const bool dww = (int)blockIdx.x < dww_blocks;
  const int b0 = dww ? (int)blockIdx.x : (int)blockIdx.x - dww_blocks, n = dww ? dww_blocks : (int)gridDim.x - dww_blocks;
  const int x = b0 & 7, b = x * (n >> 3) + min(x, n & 7) + (b0 >> 3);
  if (dww) dww_product<NTT>(da, b % dww_rows, b / dww_rows);
  else weak_product(wa, b);
}

struct BwdPlan {
  int passes, most;              // passes per set of launches; the most that this batch or a smaller one takes
  int split, rt_per_split, wsplit, kp32;
  bool weak_staged;              // weak columns staged in operand order: at most an eighth of the columns
  int x_steps;                   // steps of 16 tokens of the whole batch
  size_t a_st_bytes, part_bytes, wst_bytes, pw_bytes, xw_bytes, total;
};

// passes > 0: that many per set of launches
BwdPlan plan(const owq_layer_info_t &g, int batch, int passes = 0) {
  BwdPlan p;
  const int all_passes = (batch + kPassTokens - 1) / kPassTokens;
  // Every set of launches costs the small kernels of its own (staging, weak columns, sum; 20 us and more where the product
  // takes 15), so layers whose block pairs leave compute units free take more passes at once: 1664 -> 768 at 1017 tokens
  // 58 -> 38 us.  The product's partial results do not grow: more passes, fewer ranges of rows.  Where one set does not hold
  // them all, equal sets of more than six (10752 x 6144, 13 passes as 7 + 6: 472 -> 358 us), else four as on large layers: a short
  // last set has the others' ranges of rows and leaves the chip idle (9856 -> 6400, eight passes as 6 + 2: 255 -> 287).
  const size_t pass_bytes = (size_t)(g.n_rt + 1) * 8192;
  int most = 256 / g.nbp < kMorePasses ? 256 / g.nbp : kMorePasses;
  if (most * pass_bytes > kMoreBytes) most = (int)(kMoreBytes / pass_bytes);
  if (most < kLaunchPasses) most = kLaunchPasses;
  const int sets = (all_passes + most - 1) / most, equal = sets > 1 ? (all_passes + sets - 1) / sets : all_passes;
  p.most = all_passes < most ? all_passes : most;
  p.passes = passes > 0 ? passes : sets > 1 && equal <= 6 ? kLaunchPasses : equal < 1 ? 1 : equal;
  // Ranges of rows per block pair.  A compute unit holds one workgroup at a time, so the product takes rounds of 256
  // workgroups, each as long as its row tiles (0.7 us) and a fixed part; ranges cost a write and a read of
  // their partial results, a single one the store of dx.  In us, fitted to measurements on MI355X.
  int split = 1;
  double best = 1e30;
  for (int sp = 1; sp <= kSplitMax && sp <= g.n_rt; ++sp) {
    const long long wgs = (long long)g.nbp * sp * p.passes;
    const double rounds = (double)((wgs + 255) / 256);
    const double cost = rounds * (0.7 * ((g.n_rt + sp - 1) / sp) + 6.0) + sp * (p.passes * kPassTokens * 256.0 * g.nbp * (sp > 1 ? 8.0 : 2.0) / 4e6);
    if (cost < best) {
      best = cost;
      split = sp;
    }
  }
  p.rt_per_split = (g.n_rt + split - 1) / split;
  p.split = (g.n_rt + p.rt_per_split - 1) / p.rt_per_split;
  p.a_st_bytes = (size_t)p.passes * (g.n_rt + 1) * 2 * 4 * 64 * 16;
  p.part_bytes = p.split == 1 ? 0 : (size_t)p.passes * p.split * kPassTokens * ((size_t)g.nbp * 256) * 4;
  p.kp32 = (g.kp + 31) / 32;
  p.weak_staged = g.k > 0 && p.kp32 <= g.nbp;
  // weak columns: ranges of at least the four row tiles whose loads go out together
  p.wsplit = (g.n_rt + 3) / 4 < kWeakSplit ? (g.n_rt + 3) / 4 : kWeakSplit;
  p.wst_bytes = p.weak_staged ? (size_t)g.n_rt * 2 * p.kp32 * 64 * 16 : 0;
  p.pw_bytes = p.weak_staged ? (size_t)p.passes * p.wsplit * kPassTokens * 32 * p.kp32 * 4 : 0;
  p.x_steps = (batch + 15) / 16;
  p.xw_bytes = g.k > 0 ? (size_t)p.x_steps * p.kp32 * 64 * 16 : 0;
  p.total = p.a_st_bytes + p.part_bytes + p.wst_bytes + p.pw_bytes + p.xw_bytes;
  return p;
}

bool live(owq_handle_t h) { return h && h->magic == kMagic; }

}  // namespace

int prepare_backward_kernels(const owq_layer_info_t &g, int32_t lds_limit) {
  if (kProdLds > lds_limit) return (int)hipErrorInvalidValue;
  return (int)hipFuncSetAttribute(reinterpret_cast<const void *>(g.bits == 3 ? owq_bwd_product<3> : owq_bwd_product<4>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kProdLds);
}

}  // namespace owq

extern "C" owq_status_t owq_backward_workspace_bytes(owq_handle_t h, int32_t batch, size_t *bytes) {
  using namespace owq;
  if (!live(h)) return OWQ_ERR_HANDLE;
  if (h->info.layout != OWQ_LAYOUT_TILE) return OWQ_ERR_LAYOUT;
  if (!bytes) return OWQ_ERR_NULL;
  if (batch < 0 || batch > OWQ_MAX_BATCH) return OWQ_ERR_BATCH;
  // A plan of more passes may need less than one of fewer (fewer ranges of rows; with one range no partial results at all).  The
  // answer covers those of all smaller batches, so that a workspace for a large batch serves them too.
  const BwdPlan p = plan(h->info, batch);
  *bytes = p.total;
  for (int n = 1; n <= p.most; ++n) {
    const size_t need = plan(h->info, batch, n).total;
    if (need > *bytes) *bytes = need;
  }
  return OWQ_OK;
}

extern "C" owq_status_t owq_linear_backward(owq_handle_t h, const void *dy, const void *x, void *dx, float *dww,
                                            int32_t batch, void *workspace, size_t workspace_bytes, void *stream) {
  using namespace owq;
  if (!live(h)) return OWQ_ERR_HANDLE;
  const owq_layer_info_t &g = h->info;
  if (g.layout != OWQ_LAYOUT_TILE) return OWQ_ERR_LAYOUT;
  if (batch < 0 || batch > OWQ_MAX_BATCH) return OWQ_ERR_BATCH;
  if (batch == 0 || (!dx && !dww)) return OWQ_OK;
  if (!dy || (dww && g.k > 0 && !x) || !workspace) return OWQ_ERR_NULL;
  const BwdPlan p = plan(g, batch);
  if (workspace_bytes < p.total) return OWQ_ERR_BUFFER;
  if (((uintptr_t)dy | (uintptr_t)x | (uintptr_t)dx | (uintptr_t)dww) & 15u) return OWQ_ERR_BUFFER;
  if ((uintptr_t)workspace & 255u) return OWQ_ERR_BUFFER;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const uint8_t *blob = static_cast<const uint8_t *>(h->dev_buf);
  uint8_t *ws = static_cast<uint8_t *>(workspace);
  hipError_t err = hipSuccess;
  u32x4 *a_st = reinterpret_cast<u32x4 *>(ws);
  float *part = reinterpret_cast<float *>(ws + p.a_st_bytes);
  u32x4 *wst = p.weak_staged ? reinterpret_cast<u32x4 *>(ws + p.a_st_bytes + p.part_bytes) : nullptr;
  float *pw = p.weak_staged ? reinterpret_cast<float *>(ws + p.a_st_bytes + p.part_bytes + p.wst_bytes) : nullptr;
  u32x4 *xw_st = reinterpret_cast<u32x4 *>(ws + p.a_st_bytes + p.part_bytes + p.wst_bytes + p.pw_bytes);
  const bool want_dww = dww && g.k > 0;
  const int per_launch = p.passes * kPassTokens;
  // The first launch stages everything the call needs; later groups of passes stage their dy only.
  for (int n0 = 0; n0 < batch && err == hipSuccess && (dx || n0 == 0); n0 += per_launch) {
    const int ntok = batch - n0 < per_launch ? batch - n0 : per_launch;
    const int passes = (ntok + kPassTokens - 1) / kPassTokens;
    StageAllArgs sa = {};
    sa.dy = {static_cast<const _Float16 *>(dy), a_st, g.d_out, g.n_rt + 1, n0, batch, passes};
    sa.weak = {reinterpret_cast<const _Float16 *>(blob + g.off_weak_w), wst, g.kp, p.kp32, g.n_rt};
    sa.x = {static_cast<const _Float16 *>(x), reinterpret_cast<const int *>(blob + g.off_weak_idx), xw_st,
            g.d_in, g.k, p.kp32, batch, p.x_steps};
    const int wide_blocks = ((g.n_rt + 2) / 2) * passes;
    sa.narrow = wide_blocks < ((g.d_out & 3) == 0 ? kStageBlocks : kStageBlocksOff) ? 1 : 0;
    sa.dy_blocks = dx ? (unsigned)(sa.narrow ? 4 * wide_blocks : wide_blocks) : 0u;
    sa.weak_blocks = dx && n0 == 0 && p.weak_staged ? (unsigned)(((long long)g.n_rt * 2 * p.kp32 * 64 + 255) / 256) : 0u;
    const unsigned x_blocks = want_dww && n0 == 0 ? (unsigned)(((long long)p.x_steps * p.kp32 * 64 + 255) / 256) : 0u;
    if (sa.dy_blocks + sa.weak_blocks + x_blocks > 0)
      hipLaunchKernelGGL(owq_bwd_stage_all, dim3(sa.dy_blocks + sa.weak_blocks + x_blocks), dim3(256), 0, st, sa);
    // the small products: dww of the whole batch with the first group, dx at the weak columns with each
    const int dww_rows = (g.d_out + 31) / 32, ntt = p.kp32 <= 2 ? p.kp32 : 4;
    const int dww_blocks = want_dww && n0 == 0 ? dww_rows * ((p.kp32 + ntt - 1) / ntt) : 0;
    const int wp_blocks = dx && p.weak_staged ? p.kp32 * p.wsplit * passes : 0;
    if (dww_blocks + wp_blocks > 0) {
      const DwwArgs da = {static_cast<const _Float16 *>(dy), xw_st, dww, g.d_out, g.k, p.kp32, batch, p.x_steps};
      const WeakProdArgs wp = {a_st, wst, pw, g.n_rt, p.kp32, p.wsplit};
      hipLaunchKernelGGL(ntt == 1 ? owq_bwd_small<1> : ntt == 2 ? owq_bwd_small<2> : owq_bwd_small<4>,
                         dim3((unsigned)(dww_blocks + wp_blocks)), dim3(256), 0, st, da, wp, dww_rows, dww_blocks);
    }
    if (dx) {
      ProdArgs pa;
      pa.codes = reinterpret_cast<const u32 *>(blob + g.off_codes);
      pa.sz = reinterpret_cast<const u32 *>(blob + g.off_sz);
      pa.a_st = a_st;
      pa.part = part;
      pa.dx = p.split == 1 ? static_cast<_Float16 *>(dx) + (size_t)n0 * g.d_in : nullptr;
      pa.d_in = g.d_in;
      pa.ntok = ntok;
      pa.n_rt = g.n_rt;
      pa.nbp = g.nbp;
      pa.chunks = g.chunks;
      pa.d_out_pad = g.d_out_pad;
      pa.d_in_pad = g.nbp * 256;
      pa.blocks_per_group = g.group_size == 0 ? 0x40000000 : g.group_size / kBlockCols;
      pa.n_groups = g.n_groups;
      pa.split = p.split;
      pa.rt_per_split = p.rt_per_split;
      const dim3 grid((unsigned)(g.nbp * p.split * passes));
      hipLaunchKernelGGL(g.bits == 3 ? owq_bwd_product<3> : owq_bwd_product<4>, grid, dim3(512), kProdLds, st, pa);
      const int dense_blocks = p.split == 1 ? 0 : (g.d_in + 1023) / 1024, weak_blocks = p.weak_staged ? (g.k + 255) / 256 : 0;
      SumArgs su = {part, pw, blob + g.off_wmask, reinterpret_cast<const int *>(blob + g.off_weak_idx),
                    static_cast<_Float16 *>(dx), g.d_in, g.nbp * 256, p.split, p.wsplit, n0, ntok, g.k, p.kp32, dense_blocks};
      if (dense_blocks + weak_blocks > 0)
        hipLaunchKernelGGL(owq_bwd_sum, dim3((unsigned)(dense_blocks + weak_blocks), (unsigned)ntok), dim3(256), 0, st, su);
      if (g.k > 0 && !p.weak_staged) {
        WeakArgs wa = {static_cast<const _Float16 *>(dy), reinterpret_cast<const _Float16 *>(blob + g.off_weak_w),
                       reinterpret_cast<const int *>(blob + g.off_weak_idx), static_cast<_Float16 *>(dx),
                       g.d_out, g.d_in, g.kp, n0, ntok};
        hipLaunchKernelGGL(owq_bwd_weak, dim3((unsigned)(g.kp / 8), (unsigned)((ntok + 7) / 8)), dim3(256), 0, st, wa);
      }
    }
    err = hipGetLastError();
  }
  if (err != hipSuccess) {
    h->info.last_hip_error = (int32_t)err;
    return OWQ_ERR_HIP;
  }
  return OWQ_OK;
}
