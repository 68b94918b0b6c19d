// Quantization configuration search (paper, section "Quantization Configuration Search") for
// gfx950: for every (output row, group of input columns) a two-dimensional grid of narrowed
// ranges is tried and the step size and zero point with the least rounding error are kept.
//
// Summing every weight's error at every grid point is five vector instructions per pair, 256 points per weight.
// Nearly all points can be ruled out without it.  With c_L the highest level of a point (step size s) and m_l the
// midpoints between its levels, rounding to nearest with clamping gives
//     E = sum (w - c_L)^2 + 2 s sum_l G(m_l),      G(m) = sum min(w - m, 0)
// and G is one concave function of the group, the same for all grid points.  So the group's weights go into a
// histogram of F bins (in LDS: a count and a sum of offsets, one 64-bit integer atomic per weight), two prefix sums
// turn it into G at the bin edges, and every grid point is bounded from below by 2^bits - 1 lookups with linear
// interpolation (a chord of a concave function lies under it).  The point with the least bound is evaluated in full,
// and then those whose bound, less a bound on its own rounding, does not exceed the least error found: one or two
// different points in all.  These evaluations take the same binary32 decisions per weight as the
// plain search and share their sums among the lanes; points whose sums come out too close to tell are summed again in
// the order of the columns, so that the choice is that of the plain search.
// Bound by vector instructions, and by how many waves a SIMD holds to issue them: a wave issues one every four or five cycles, the
// SIMD takes more.  16384 x 4096, 3-bit, groups of 128, 16 x 16 points: plain search 1780 us, four points per lane 620 (815
// instructions per group), the grid by diagonals with the general way in the same kernel 395 (five waves per SIMD), in a
// kernel of its own 357 (504; eight).  5120 x 5120, 4-bit, one scale per row: 134 -> 98 us when a wave's registers went from 227 to 112
// (two waves per SIMD -> four: columns and masks of all weights had been kept in registers from one row to the next, and masks
// in spilled scalar registers), 76 to 98 with a row per workgroup, one of several equal points of a diagonal evaluated and
// two points at a time summed in order (by whether one of the last rows has such points: 20 us); 4096 rows of 13824: 290 -> 123.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "owq.h"

namespace owq {
namespace {

typedef unsigned int u32;
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;            // waves per workgroup, each with its own LDS area
constexpr int kChunk = 1024;         // columns moved through LDS at a time
constexpr int zero_points(int bits) { return bits == 3 ? 4 : 7; }      // longest run of them that a lane takes on a diagonal
constexpr uint16_t kLeft = 0xffffu;  // as a step size: this group is left to the general grid's kernel
constexpr u32 kLeastStep = 0x38800000u;    // 2^-14 in binary32
constexpr int kMaskBytesMax = 47 * 1024;   // LDS left for the weak-column bit mask of a row: 64 KiB less the kernel's static 16.1 KiB

struct SearchArgs {
  const _Float16 *w;
  const int *weak_idx;
  uint16_t *scale, *zero;
  uint8_t *codes;
  float *err;
  int *choice;
  int d_in, g, n_groups, k, n_lo, n_hi, units, units_per_wave;
  int vec;                             // rows and groups on the grid of the lanes' runs of columns
  float qmax, shrink;
};

struct Cand {
  float s, inv, a, b;                // step size, its reciprocal, -z, qmax - z
};

// op over the 64 lanes of the wave, every lane gets the result: four steps inside the rows of
// 16 lanes on the data-parallel path, then the four row results through scalar registers
template <class T, class F>
__device__ __forceinline__ T wave_all(T v, F op) {
  auto dpp = [](T x, auto ctrl) __attribute__((always_inline)) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  v = op(v, dpp(v, std::integral_constant<int, 0xB1>{}));    // lanes ^ 1
  v = op(v, dpp(v, std::integral_constant<int, 0x4E>{}));    // lanes ^ 2
  v = op(v, dpp(v, std::integral_constant<int, 0x141>{}));   // mirror in 8
  v = op(v, dpp(v, std::integral_constant<int, 0x140>{}));   // mirror in 16
  const int i = __builtin_bit_cast(int, v);
  const T r0 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(i, 0)), r1 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(i, 16));
  const T r2 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(i, 32)), r3 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(i, 48));
  return op(op(r0, r1), op(r2, r3));
}

// Least (greatest) of the 64 lanes' values, none of them a NaN.  Written as instructions: from fminf the compiler makes four per
// step (old value, move across lanes, canonicalise, minimum) where one does.  s_nop: two wait states before a value that was
// just written is read across lanes, inside the blocks and around them, and before scalar registers that v_readlane wrote are
// used: the compiler, which adds these between its own instructions, does not look into a block.
__device__ __forceinline__ float wave_min(float v) {
  asm("s_nop 1\n\tv_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_min_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1"
      : "+v"(v));
  const int i = __builtin_bit_cast(int, v);
  const int r0 = __builtin_amdgcn_readlane(i, 0), r1 = __builtin_amdgcn_readlane(i, 16), r2 = __builtin_amdgcn_readlane(i, 32);
  float m = __builtin_bit_cast(float, __builtin_amdgcn_readlane(i, 48));
  asm("s_nop 1\n\tv_min_f32 %0, %1, %0\n\tv_min_f32 %0, %2, %0\n\tv_min_f32 %0, %3, %0\n\ts_nop 1" : "+v"(m) : "s"(r0), "s"(r1), "s"(r2));
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, m)));
}
__device__ __forceinline__ float wave_max(float v) { return -wave_min(-v); }

// Step size, reciprocal and zero point of the grid point that cuts the fractions fa and fb of
// the range from its ends.  Every operation is a single binary32 operation in the order the
// interface states; nothing may be fused here.
// ANY: ranges that are no numbers too.  Otherwise the two divisions take three instructions each instead of ten, with
// the same results: the quotient by 7 or 15 and the reciprocal of an fp16 number, corrected by their residuals, were
// compared with the divisions for every mantissa.
template <bool ANY>
__device__ __forceinline__ Cand candidate(float lo, float hi, float fa, float fb, float qmax, float rqmax) {
#pragma clang fp contract(off)
  const float r = hi - lo;
  const float pa = fa * r, pb = fb * r;
  const float lo_i = lo + pa, hi_j = hi - pb;
  const float width = hi_j - lo_i;
  float s32;
  if (ANY) {
    s32 = width / qmax;
  } else {
    const float q0 = width * rqmax;
    s32 = __builtin_fmaf(__builtin_fmaf(-q0, qmax, width), rqmax, q0);
  }
  s32 = s32 > 0x1p-14f ? s32 : 0x1p-14f;
  const float s = (float)(_Float16)s32;
  float inv;
  if (ANY) {
    inv = 1.0f / s;
  } else {
    const float r0 = __builtin_amdgcn_rcpf(s);
    inv = __builtin_fmaf(__builtin_fmaf(-s, r0, 1.f), r0, r0);
  }
  const float zl = -lo_i * inv;
  float z = __builtin_rintf(zl);
  z = z < -2048.f ? -2048.f : (z > 2048.f ? 2048.f : z);
  Cand c;
  c.s = s;
  c.inv = inv;
  c.a = 0.f - z;                     // 0 - z: no negative zero
  c.b = qmax - z;
  return c;
}

// The step size of a range of this width, as candidate<false> finds it.
__device__ __forceinline__ float step_of(float width, float qmax, float rqmax) {
#pragma clang fp contract(off)
  const float q0 = width * rqmax;
  const float s32 = __builtin_fmaf(__builtin_fmaf(-q0, qmax, width), rqmax, q0);
  return (float)(_Float16)(s32 > 0x1p-14f ? s32 : 0x1p-14f);
}
// its reciprocal, and the zero point of a range that starts at lo_i
__device__ __forceinline__ float reciprocal(float s) {
  const float r0 = __builtin_amdgcn_rcpf(s);
  return __builtin_fmaf(__builtin_fmaf(-s, r0, 1.f), r0, r0);
}
__device__ __forceinline__ float zero_of(float lo_i, float inv) {
#pragma clang fp contract(off)
  return __builtin_amdgcn_fmed3f(__builtin_rintf(-lo_i * inv), -2048.f, 2048.f);
}
__device__ __forceinline__ float cut_lo(float lo, float f, float r) {
#pragma clang fp contract(off)
  const float p = f * r;
  return lo + p;
}
__device__ __forceinline__ float cut_hi(float hi, float f, float r) {
#pragma clang fp contract(off)
  const float p = f * r;
  return hi - p;
}

// fraction of the range that grid point i of n cuts: binary32 of (shrink * i) / (n - 1) in binary64
__device__ __forceinline__ float cut_fraction(float shrink, int i, int n) {
  if (n == 1) return 0.f;
  return (float)((double)shrink * (double)i / (double)(n - 1));
}

__device__ __forceinline__ void wave_lds_fence() {
  // LDS serves one wave's instructions in order; this keeps the compiler from moving them
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ bool is_weak(const u32 *mask, int col) {
  return ((mask[col >> 5] >> (col & 31)) & 1u) != 0u;
}

// Moves the non-weak weights of columns [col0, col0 + n) of a row into `list` as fp32, in
// order, and returns how many there are.  n <= kChunk.
__device__ __forceinline__ int stage(const _Float16 *wrow, int col0, int n, float *list, const u32 *mask, int lane) {
  int cnt = 0;
  for (int t = 0; t < n; t += 64) {
    const int c = t + lane;
    const bool valid = c < n;
    const float v = valid ? (float)wrow[col0 + c] : 0.f;
    const bool keep = valid && !is_weak(mask, col0 + c);
    const unsigned long long m = __ballot(keep);
    const int pos = cnt + (int)__builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
    if (keep) list[pos] = v;
    cnt += __builtin_popcountll(m);
  }
  wave_lds_fence();
  return cnt;
}

template <int CPL>
__device__ __forceinline__ void accumulate(const Cand (&cd)[CPL], float (&e)[CPL], float w) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const float t = w * cd[c].inv;
    const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(t), cd[c].a, cd[c].b);   // q - z
    const float d = __builtin_fmaf(-cd[c].s, q, w);
    e[c] = __builtin_fmaf(d, d, e[c]);
  }
}

// What the search of one (row, group) yields.
struct Best {
  float s, inv, z, e;
  int id;
};

// Widens a zero-width range to reach 0; true if there is nothing to search.
__device__ __forceinline__ bool degenerate(float &lo, float &hi, int kept) {
  if (kept == 0) return true;
  if (hi == lo) {
    lo = lo < 0.f ? lo : 0.f;
    hi = hi > 0.f ? hi : 0.f;
    return hi == lo;
  }
  return false;
}

__device__ __forceinline__ void store_choice(const SearchArgs &a, int row, int gi, const Best &b, int lane) {
  if (lane == 0) {
    const size_t o = (size_t)row * a.n_groups + gi;
    a.scale[o] = __builtin_bit_cast(uint16_t, (_Float16)b.s);
    a.zero[o] = __builtin_bit_cast(uint16_t, (_Float16)b.z);
    if (a.err != nullptr) a.err[o] = b.e;
    if (a.choice != nullptr) a.choice[o] = b.id;
  }
}

__device__ __forceinline__ uint8_t code_of(float v, const Best &b, float qmax) {
  const float za = 0.f - b.z, zb = qmax - b.z;
  return (uint8_t)(int)(__builtin_amdgcn_fmed3f(__builtin_rintf(v * b.inv), za, zb) - za);
}

// ---------------------------------------------------------------------------
// bounds from a histogram
// ---------------------------------------------------------------------------
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp0(int v) {       // 0 in lanes without a source
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
// sum over the lanes up to and including this one
__device__ __forceinline__ int scan_lanes(int v) {
  v += dpp0<0x111, 0xf>(v);
  v += dpp0<0x112, 0xf>(v);
  v += dpp0<0x114, 0xf>(v);
  v += dpp0<0x118, 0xf>(v);
  v += dpp0<0x142, 0xa>(v);
  v += dpp0<0x143, 0xc>(v);
  return v;
}
__device__ __forceinline__ float scan_lanes(float v) {
  auto f = [](int x) __attribute__((always_inline)) { return __builtin_bit_cast(float, x); };
  auto i = [](float x) __attribute__((always_inline)) { return __builtin_bit_cast(int, x); };
  v += f(dpp0<0x111, 0xf>(i(v)));
  v += f(dpp0<0x112, 0xf>(i(v)));
  v += f(dpp0<0x114, 0xf>(i(v)));
  v += f(dpp0<0x118, 0xf>(i(v)));
  v += f(dpp0<0x142, 0xa>(i(v)));
  v += f(dpp0<0x143, 0xc>(i(v)));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_all(v, [](float x, float y) { return x + y; });
}

// The search of groups of at most 64 TW NT columns by a team of TW waves (1 or 4, one or four teams per workgroup).
// Lane t of the team keeps its NT weights of a group in registers, V neighbouring columns at a time; they give
// the range, the histogram, the evaluations and the codes: one global read per weight.
// Bins: 4 per lane of the team.  256 for a wave (groups of at most 1024: the bounds are within 0.7 % at 3 bits and
// groups of 128, 512 bins would leave 4 points instead of 5 and cost a longer scan), 1024 for four waves.
template <int TW, int NT, int POINTS>
struct Team {
  static constexpr int V = NT < 8 ? NT : 8;
  static constexpr int LANES = 64 * TW;
  static constexpr int F = 4 * LANES;
  static constexpr int CPL = POINTS;               // grid points per lane: at most 64 TW POINTS of them
  static __device__ __forceinline__ int column(int t, int lane) { return ((t / V) * LANES + lane) * V + t % V; }
};

// Table entry b + 1: G at bin b's lower edge and its increase over the bin; entries 0 and F + 1 continue G one bin beyond
// the range on either side, which is as far as the midpoints of a grid point get unless its step size or zero point
// was clamped (those are evaluated in full).
struct Knot {
  float g, dg;
};

__device__ __forceinline__ unsigned long long uniform(unsigned long long v) {
  return ((unsigned long long)(u32)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (u32)__builtin_amdgcn_readfirstlane((int)v);
}

// What the waves of a team of four exchange.
struct TeamShared {
  Cand cand[256];
  float part[256][4];
  float wave[4][4];
  unsigned long long alive[4];
  int scan_i[4];
  float scan_f[4];
};

//
// BITS > 0 (a wave per group, as many points at either end): on a diagonal i + j of the grid the width is one value but for
// rounding, so all its points have one step size, and their zero points are a short run of integers: of 256 points about 107
// (3 bits) are different ones, and those of one diagonal share all midpoints but a few.  Two lanes take a diagonal, half of
// its points each; L levels and Z zero points need L + Z - 1 lookups, of which every L in a row are a grid point's (3 bits: 10
// lookups where four points per lane took 28).  Z covers the runs of the square grids that come here.  A group where a diagonal
// has more than one step size (the widths' rounding straddles a binary16 boundary, inside a half or between the two), where a
// run is longer all the same, a step size is at its least value, a midpoint lies beyond the table or three errors are too close
// to tell is marked in `scale` (kLeft).
// BITS < 0: the general grid for what is marked.  In a kernel of its own since the general way takes 30 registers more: 107 ->
// 90 us for the 2^17 groups of 128 of a 4096 x 4096 matrix, and 5 us for the launch that looks for marks.
template <int TW, int NT, int POINTS, int BITS>
__global__ __launch_bounds__(256, NT <= 4 ? 5 : NT <= 24 ? 4 : 2) void owq_search_bounds(const SearchArgs a) {
  using T = Team<TW, NT, POINTS>;
  constexpr int V = T::V, LANES = T::LANES, F = T::F, CPL = T::CPL, TEAMS = 4 / TW;
  __shared__ __attribute__((aligned(16))) unsigned long long hist[TEAMS][F + 2];
  __shared__ TeamShared sh[1];                     // four waves only
  extern __shared__ u32 mask[];                    // bit c = column c is weak; (d_in + 31) / 32 words
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int tl = TW == 4 ? tid : lane;             // lane within the team
  unsigned long long *bins = hist[TW == 4 ? 0 : wv];
  const int team = TW == 4 ? (int)blockIdx.x : (int)blockIdx.x * 4 + wv;
  const int u0 = team * a.units_per_wave;
  int n_units = a.units - u0 < a.units_per_wave ? a.units - u0 : a.units_per_wave;         // same for the team
  unsigned long long todo = 0ull;                  // BITS < 0: which of this wave's 64 or fewer groups
  if constexpr (BITS < 0) {
    todo = __ballot(lane < n_units && a.scale[u0 + (lane < n_units ? lane : 0)] == kLeft);
    if (__syncthreads_or(todo != 0ull) == 0) return;
    n_units = __builtin_popcountll(todo);
  }
  for (int i = tid; i < (a.d_in + 31) >> 5; i += 256) mask[i] = 0u;
  __syncthreads();
  for (int p = tid; p < a.k; p += 256) {
    const u32 c = (u32)a.weak_idx[p];
    if (c < (u32)a.d_in) atomicOr(&mask[c >> 5], 1u << (c & 31));
  }
  __syncthreads();
  const int ncand = a.n_lo * a.n_hi;
  float fa[CPL], fb[CPL];
  auto cuts = [&](int l) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int id = l + LANES * c;
      const int i = id / a.n_hi, j = id - i * a.n_hi;
      fa[c] = cut_fraction(a.shrink, i < a.n_lo ? i : 0, a.n_lo);
      fb[c] = cut_fraction(a.shrink, j, a.n_hi);
    }
  };
  if constexpr (BITS <= 0) cuts(tl);
  // what follows from the value is worked out where it is used: kept out of the registers of the rest
  auto seldom = [](auto l) __attribute__((always_inline)) {
    asm volatile("" : "+v"(l));
    return l;
  };
  // a lane's half of a diagonal: its first and last point (i, d - i), and their cuts
  float f0a = 0.f, f0b = 0.f, f1a = 0.f, ft = 0.f;
  auto half_of = [&](int l, int &i0, int &i1, int &j0) __attribute__((always_inline)) {
    const int m = a.n_hi - 1, d = min(l >> 1, 2 * m), i_min = max(0, d - m), i_max = min(d, m), h0 = (i_max - i_min + 2) >> 1;
    i0 = l & 1 ? min(i_min + h0, i_max) : i_min;
    i1 = l & 1 ? i_max : i_min + h0 - 1;
    j0 = d - i0;
  };
  if constexpr (BITS > 0) {
    int i0, i1, j0;
    half_of(lane, i0, i1, j0);
    f0a = cut_fraction(a.shrink, i0, a.n_hi);
    f0b = cut_fraction(a.shrink, j0, a.n_hi);
    f1a = cut_fraction(a.shrink, i1, a.n_hi);
    ft = cut_fraction(a.shrink, min(lane, a.n_hi - 1), a.n_hi);
  }
  if (n_units <= 0) return;                        // four waves: the whole workgroup
  int row = u0 / a.n_groups, gi = u0 - row * a.n_groups;
  auto team_barrier = [&]() __attribute__((always_inline)) {
    if constexpr (TW == 4) __syncthreads();
    else wave_lds_fence();
  };

  // columns past the end of a short last group are fetched from its last ones and dropped
  auto fetch = [&](_Float16 (&dst)[NT], int r, int g) __attribute__((always_inline)) {
    const int c0 = g * a.g, len = a.d_in - c0 < a.g ? a.d_in - c0 : a.g;
    const _Float16 *src = a.w + (size_t)r * a.d_in + c0;
    typedef _Float16 hv __attribute__((ext_vector_type(V)));
    if (a.vec) {                                   // rows on the grid of V elements, len a multiple of V
#pragma unroll
      for (int t = 0; t < NT; t += V) {
        const int c = T::column(t, tl);
        const hv v = *reinterpret_cast<const hv *>(src + (c < len ? c : len - V));
#pragma unroll
        for (int e = 0; e < V; ++e) dst[t + e] = v[e];
      }
    } else {
      const int l = seldom(tl);                    // or the columns of all weights stay in registers
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int c = T::column(t, l);
        dst[t] = src[c < len ? c : len - 1];
      }
    }
  };
  // four waves: the grid point before this thread's on its diagonal, which has the same width
  const int before = TW == 4 && tid < ncand && tid >= a.n_hi && (tid + 1) % a.n_hi != 0 ? tid - (a.n_hi - 1) : -1;
  // a wave fetches its next group while it searches one; with four waves to a row other workgroups fill the wait
  constexpr bool kAhead = TW == 1 && BITS >= 0;
  float cur[NT];
  _Float16 nxt[NT];
  if (BITS >= 0) fetch(nxt, row, gi);
  for (int uu = 0; uu < n_units; ++uu) {
    if constexpr (BITS < 0) {
      const int u = u0 + __builtin_ctzll(todo);
      todo &= todo - 1;
      row = u / a.n_groups;
      gi = u - row * a.n_groups;
    }
    const int c0 = gi * a.g;
    const int len = a.d_in - c0 < a.g ? a.d_in - c0 : a.g;
    int nrow = row, ngi = gi + 1;
    if (ngi == a.n_groups) {
      ngi = 0;
      ++nrow;
    }
    if (!kAhead && (BITS < 0 || uu > 0)) fetch(nxt, row, gi);
#pragma unroll
    for (int t = 0; t < NT; ++t) cur[t] = (float)nxt[t];
    if (kAhead && uu + 1 < n_units) fetch(nxt, nrow, ngi);
    // ---- range; an empty histogram ----
    std::conditional_t<(NT > 32), unsigned long long, u32> kept = 0;     // bit t: weight t of this lane takes part
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int t = 0; t < NT; t += V) {
      const int c = T::column(t, tl);
      u32 m = 0u;
      if (c < len) {
        m = ~(mask[(c0 + c) >> 5] >> ((c0 + c) & 31)) & ((1u << V) - 1u);
        if (len - c < V) m &= (1u << (len - c)) - 1u;
      }
      kept |= (decltype(kept))m << t;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const u32 v = __builtin_bit_cast(u32, cur[t + e]), in = (u32)__builtin_amdgcn_sbfe((int)m, e, 1);      // all ones or none
        lo = __builtin_fminf(lo, __builtin_bit_cast(float, (in & v) | (~in & 0x7f800000u)));      // ignores what is no number
        hi = __builtin_fmaxf(hi, __builtin_bit_cast(float, (in & v) | (~in & 0xff800000u)));
        cur[t + e] = __builtin_bit_cast(float, in & v);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) bins[tl * 4 + i] = 0ull;
    lo = wave_min(lo);
    hi = wave_max(hi);
    bool any = __ballot(kept != 0) != 0ull;
    if constexpr (TW == 4) {
      if (lane == 0) {
        sh[0].wave[wv][0] = lo;
        sh[0].wave[wv][1] = hi;
        sh[0].wave[wv][2] = any ? 1.f : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float l = sh[0].wave[i][0], h = sh[0].wave[i][1];
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
        any |= sh[0].wave[i][2] != 0.f;
      }
    } else {
      wave_lds_fence();
    }
    const bool nothing = degenerate(lo, hi, any ? 1 : 0);
    Best best = {1.f, 1.f, 0.f, 0.f, 0};
    bool left = false;                             // for the general grid's kernel
    if (!nothing) {
      // error of grid point (s, inv, za, zb) over this lane's weights, over the wave
      auto evaluate = [&](const Cand &p) __attribute__((always_inline)) {
        float e = 0.f;
        // 0 is a level: what does not take part, held as 0, adds nothing.  (Few weights: a branch costs more than their masks.)
        if (NT >= 8 && p.a <= 0.f && p.b >= 0.f) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(cur[t] * p.inv), p.a, p.b);   // q - z
            const float d = __builtin_fmaf(-p.s, q, cur[t]);
            e = __builtin_fmaf(d, d, e);
            if (NT >= 16 && t % 8 == 7) __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          const auto in = NT >= 8 ? seldom(kept) : kept;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(cur[t] * p.inv), p.a, p.b);
            const float d = (in >> t) & 1u ? __builtin_fmaf(-p.s, q, cur[t]) : 0.f;
            e = __builtin_fmaf(d, d, e);
            if (NT >= 16 && t % 8 == 7) __builtin_amdgcn_sched_barrier(0);
          }
        }
        return wave_sum(e);
      };
      const float idelta = (float)F * __builtin_amdgcn_rcpf(hi - lo);      // bins per unit, to a unit in the last place
      // ---- histogram: count in the upper half, sum of the offsets inside the bin (in 2^-16 bins) in the lower ----
      float s2 = 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float u = (cur[t] - lo) * idelta;
        const int b = (int)__builtin_amdgcn_fmed3f(u, 0.f, (float)(F - 1));
        const float f = u - (float)b;
        const float uc = u - (float)(F / 2);
        const u32 off = (u32)__builtin_fmaf(f, 65536.f, 0.5f);
        if constexpr (NT >= 8) {                   // adds nothing for what does not take part: no branch per weight
          const u32 in = (u32)__builtin_amdgcn_sbfe((int)(u32)(kept >> (t & 32)), t & 31, 1);
          const float ui = __builtin_bit_cast(float, in & __builtin_bit_cast(u32, uc));
          atomicAdd(&bins[b], ((unsigned long long)(in & 1u) << 32) | (unsigned long long)(in & off));
          s2 = __builtin_fmaf(ui, ui, s2);
          if (NT >= 16 && t % 8 == 7) __builtin_amdgcn_sched_barrier(0);      // or all weights' operands are in registers at once
        } else if ((kept >> t) & 1u) {
          atomicAdd(&bins[b], (1ull << 32) | (unsigned long long)off);
          s2 = __builtin_fmaf(uc, uc, s2);
        }
      }
      s2 = wave_sum(s2);
      team_barrier();
      // ---- G at the edges: the increase over bin b is -(weights below it) - (weights in it - their offsets) ----
      unsigned long long h[4];
      int n4 = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h[i] = bins[tl * 4 + i];
        n4 += (int)(h[i] >> 32);
      }
      const int incl = scan_lanes(n4);
      int cnt = __builtin_amdgcn_readlane(incl, 63);           // weights that take part
      float dg[4], d4 = 0.f;
      int upto = incl - n4;                        // weights up to the bin's upper edge
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        upto += (int)(h[i] >> 32);
        dg[i] = __builtin_fmaf((float)(u32)h[i], 0x1p-16f, -(float)upto);
        d4 = i == 0 ? dg[0] : d4 + dg[i];
      }
      const float ginc = scan_lanes(d4);
      float g = ginc - d4, wbelow = 0.f;         // of the wave's own bins; weights in the waves before
      if constexpr (TW == 4) {
        if (lane == 63) {
          sh[0].scan_i[wv] = incl;
          sh[0].scan_f[wv] = ginc;
        }
        if (lane == 0) sh[0].wave[wv][0] = s2;
        __syncthreads();
        s2 = (sh[0].wave[0][0] + sh[0].wave[1][0]) + (sh[0].wave[2][0] + sh[0].wave[3][0]);
        cnt = (sh[0].scan_i[0] + sh[0].scan_i[1]) + (sh[0].scan_i[2] + sh[0].scan_i[3]);
        float goff = 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (i < wv) {
            goff += sh[0].scan_f[i] - wbelow * 256.f;
            wbelow += (float)sh[0].scan_i[i];
          }
        g += goff - wbelow * (float)(lane * 4);
      }
      Knot *knot = reinterpret_cast<Knot *>(bins);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d = dg[i] - wbelow;
        knot[tl * 4 + i + 1] = Knot{g, d};
        g += d;
      }
      if (tl == 0) knot[0] = Knot{0.f, 0.f};
      if (tl == LANES - 1) knot[F + 1] = Knot{g, -(float)cnt};
      team_barrier();
      const float gend = knot[F + 1].g, n = (float)cnt;
      const float s1 = gend + n * (float)(F / 2);            // sum of the centred weights
      const bool any_odd = !(s2 < INFINITY);       // a weight that is no number: the table says nothing
      // ---- bounds ----
      // What rounding can do to a value: eight operations on terms of at most `mag`, and positions (midpoints, levels)
      // that are off by `eps` bins, each seen by all weights
      const float far = __builtin_fmaxf(__builtin_fabsf(lo), __builtin_fabsf(hi)) * idelta, half = (float)(F / 2);
      const float mag = 2.f * (s2 + half * (half * n + 2.f * __builtin_fabsf(s1)));
      const float eps = (BITS > 0 ? 5.f : 3.f) * (float)F + 2.f * far;
      const float slack = 0x1p-24f * (8.f * mag + 4.f * n * (float)F * eps);
      const float to_bins = any_odd ? 1.f : idelta * idelta * (1.f + 0x1p-12f);
      // errors this close may change places: four deviations of the rounding of two sums of cnt terms (0.3 sqrt(cnt / 3) units in
      // the 24th place each)
      const float close = 1.f + 0x1p-24f * (__builtin_amdgcn_sqrtf((float)cnt) + 8.f);
      auto lane_of = [&](float v, int src) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
      };
      // The error of a grid point as one sum in the order of the columns, which is what ranks points whose errors agree to
      // the rounding of such sums: the residuals go through LDS (where the bins were), the sum runs on every lane.
      auto residual = [&](const Cand &p, int t) __attribute__((always_inline)) {
        const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(cur[t] * p.inv), p.a, p.b);
        return (seldom(kept) >> t) & 1u ? __builtin_fmaf(-p.s, q, cur[t]) : 0.f;
      };
      float *res = reinterpret_cast<float *>(bins);
      auto add4 = [](float e, f4v d) __attribute__((always_inline)) {
        return __builtin_fmaf(d[3], d[3], __builtin_fmaf(d[2], d[2], __builtin_fmaf(d[1], d[1], __builtin_fmaf(d[0], d[0], e))));
      };
      auto in_order = [&](const Cand &p) __attribute__((always_inline)) {           // one wave
        float e = 0.f;
#pragma unroll
        for (int t0 = 0; t0 < NT; t0 += V) {
          wave_lds_fence();
#pragma unroll
          for (int t = t0; t < t0 + V; ++t) res[lane * V + t - t0] = residual(p, t);
          wave_lds_fence();
          const int n4 = min(V * 64, (len - t0 * 64 + 3) & ~3) >> 2;
#pragma unroll 4
          for (int i = 0; i < n4; ++i) e = add4(e, reinterpret_cast<const f4v *>(res)[i]);
        }
        return e;
      };
      if constexpr (BITS > 0) {
        bool found = false;
        constexpr int L = (1 << BITS) - 1, Z = zero_points(BITS);
        const float qmax = (float)L, rqmax = 1.f / (float)L;
        const float r = hi - lo, lo0 = cut_lo(lo, f0a, r), width = cut_hi(hi, f0b, r) - lo0;
        // no point's width is further from another's than 5.6 2^-24 (r + largest end): seven roundings each
        const float tol = 0x1p-21f * (r + __builtin_fmaxf(__builtin_fabsf(lo), __builtin_fabsf(hi)));
        const float s = step_of(width, qmax, rqmax);
        const float lo_t = cut_lo(lo, ft, r);
        bool other = !(s > 0x1p-14f);
        if (__ballot(step_of(width - tol, qmax, rqmax) != step_of(width + tol, qmax, rqmax)) != 0ull) {
          const float hi_t = cut_hi(hi, ft, r);
          int i0, i1, j0;
          half_of(seldom(lane), i0, i1, j0);
          // the diagonal's other half, of which this lane's points say nothing; then this half point by point
          other |= __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, s), 0xB1, 0xf, 0xf, true)) != s;
#pragma unroll 1
          for (int p = 1; p < 8; ++p) {
            const int o = min(p, i1 - i0);
            other |= step_of(__shfl(hi_t, j0 - o) - __shfl(lo_t, i0 + o), qmax, rqmax) != s;
          }
        }
        const float inv = reciprocal(s), su = s * idelta;
        const float z0 = zero_of(lo0, inv), z1 = zero_of(cut_lo(lo, f1a, r), inv), span = z0 - z1;
        const float p1 = (s * (0.5f - z0) - lo) * idelta + 1.f;
        other |= !(span <= (float)(Z - 1)) || !(p1 >= 0.f) || !(__builtin_fmaf(span + (float)(L - 1), su, p1) < (float)(F + 2));
        if (!any_odd && __ballot(other) == 0ull) {
          float v[L + Z - 1];                      // G at the midpoints of the run
          float core = 0.f;                        // sum of those that all its zero points have
          constexpr int AT_ONCE = BITS == 3 ? 5 : 7;     // reads in flight
#pragma unroll
          for (int t0 = 0; t0 < L + Z - 1; t0 += AT_ONCE) {
            Knot k[AT_ONCE];
            float f[AT_ONCE];
#pragma unroll
            for (int t = 0; t < AT_ONCE; ++t) {
              float p = __builtin_fmaf((float)(t0 + t), su, p1);
              if (t0 + t >= L) p = __builtin_fminf(p, (float)(F + 1));      // not of this lane's zero points
              k[t] = knot[(u32)p];
              f[t] = __builtin_amdgcn_fractf(p);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < AT_ONCE; ++t) {
              v[t0 + t] = __builtin_fmaf(f[t], k[t].dg, k[t].g);
              if (t0 + t >= Z - 1 && t0 + t < L) core += v[t0 + t];
            }
          }
          float gs[Z];                             // sums of L in a row: what comes before those, and after
          gs[Z - 1] = core;
#pragma unroll
          for (int k = Z - 2; k >= 0; --k) gs[k] = gs[k + 1] + v[k];
          float after = 0.f;
#pragma unroll
          for (int k = 1; k < Z; ++k) {
            after += v[L + k - 1];
            gs[k] += after;
          }
          const float top = (s * (qmax - z0) - lo) * idelta - half;
          // the halves' runs often meet in one zero point, which the first half has
          const float z1_first = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, z1), 0xA0, 0xf, 0xf, true));
          const bool live = lane < 4 * a.n_hi - 2;
          float bound[Z];
#pragma unroll
          for (int k = 0; k < Z; ++k) {
            const float tk = __builtin_fmaf((float)k, su, top);
            const float e = __builtin_fmaf(2.f * su, gs[k], __builtin_fmaf(tk, __builtin_fmaf(tk, n, -2.f * s1), s2)) - slack;
            const bool is = live && (k == 0 ? !((lane & 1) && z0 == z1_first) : (float)k <= span);
            bound[k] = is ? e : INFINITY;
          }
          // the point with the least bound, then the next one until bounds exceed the least error found
          best.e = INFINITY;
          Best second = best;                      // and the next best, and the third one's error
          float third = INFINITY;
          const float lim = to_bins * close;
          for (;;) {
            float mine = bound[0];
#pragma unroll
            for (int k = 1; k < Z; ++k) mine = __builtin_fminf(mine, bound[k]);
            if (__ballot(mine <= best.e * lim && mine < INFINITY) == 0ull) break;
            const float wl = wave_min(mine);
            const unsigned long long at = __ballot(mine == wl);
            if (at == 0ull) break;
            const int src = __builtin_ctzll(at);
            float kz = 0.f;                        // which of the lane's zero points
            bool due = lane == src;
#pragma unroll
            for (int k = 0; k < Z; ++k) {
              const bool this_one = due && bound[k] == wl;
              kz = this_one ? (float)k : kz;
              bound[k] = this_one ? INFINITY : bound[k];
              due = due && !this_one;
            }
            Cand p;
            p.s = lane_of(s, src);
            p.inv = lane_of(inv, src);
            const float z = lane_of(z0 - kz, src);
            p.a = 0.f - z;
            p.b = qmax - z;
            // the points of the diagonal with this zero point; none where they step over it
            const int d = src >> 1, ia = max(0, d - (a.n_hi - 1)), ib = min(d, a.n_hi - 1);
            const unsigned long long of = __ballot(zero_of(lo_t, p.inv) == z) & (((2ull << ib) - 1ull) & ~((1ull << ia) - 1ull));
            if (of == 0ull) continue;
            const int i = __builtin_ctzll(of), id = i * a.n_hi + d - i;
            const Best b = {p.s, p.inv, 0.f - p.a, evaluate(p), id};      // no negative zero
            third = __builtin_fminf(third, __builtin_fmaxf(b.e, second.e));
            const bool better = b.e < best.e || (b.e == best.e && id < best.id);
            if (better || b.e < second.e) second = better ? best : b;
            if (better) best = b;
          }
          const float near = best.e * close;
          found = best.e < INFINITY && !(best.e > 0.f && third <= near);
          if (found && best.e > 0.f && second.e <= near) {       // two that are too close to tell
            best.e = in_order(Cand{best.s, best.inv, 0.f - best.z, qmax - best.z});
            second.e = in_order(Cand{second.s, second.inv, 0.f - second.z, qmax - second.z});
            if (second.e < best.e || (second.e == best.e && second.id < best.id)) best = second;
          }
        }
        left = !found;
      }
      if constexpr (BITS <= 0) {
        Cand cd[CPL];
        float bound[CPL];
        float least = INFINITY;                      // least value (not bound) from the table, and its grid point
        int first = 0x7fffffff;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          cd[c] = candidate<false>(lo, hi, fa[c], fb[c], a.qmax, 1.f / a.qmax);
          bound[c] = -INFINITY;
        }
        if (any_odd) {
#pragma unroll
          for (int c = 0; c < CPL; ++c) cd[c] = candidate<true>(lo, hi, fa[c], fb[c], a.qmax, 0.f);
        } else {
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            const float su = cd[c].s * idelta, top = (cd[c].s * cd[c].b - lo) * idelta - half;
            const float p1 = (cd[c].s * (cd[c].a + 0.5f) - lo) * idelta + 1.f;
            const bool inside = p1 >= 0.f && __builtin_fmaf(a.qmax - 1.f, su, p1) < (float)(F + 2);
            float gs = 0.f;
            if (inside) {
#pragma unroll
              for (int l = 0; l < 15; ++l) {
                if (l == 7 && a.qmax < 15.f) break;
                const float p = __builtin_fmaf((float)l, su, p1);
                const Knot k = knot[(u32)p];
                gs = __builtin_fmaf(__builtin_amdgcn_fractf(p), k.dg, gs + k.g);
              }
            }
            const float sq = __builtin_fmaf(top, __builtin_fmaf(top, n, -2.f * s1), s2);
            const float e = __builtin_fmaf(2.f * su, gs, sq);
            const int id = tl + LANES * c;
            const bool is = id < ncand;
            bound[c] = is ? (inside ? e - slack : -INFINITY) : INFINITY;
            if (is && inside && e < least) {
              least = e;
              first = id;
            }
          }
        }
        // Four waves: waves 0 and 1 sum two points, whose residuals come 1024 columns (two waves' runs of them) at a time.  A chain of
        // dependent additions is all latency: 28 of a wave's 32 values in registers are still to be added when one is read, and
        // the wave goes first on its SIMD.  (One point after the other, a chain of LDS reads each, took 87 us per point on a row
        // of 5120 columns; 512 columns of four points, 16 values ahead: 8 us more for a matrix of 5120 rows with a few of these.)
        auto in_order2 = [&](int id0, int id1) __attribute__((always_inline)) {
          float e = 0.f;
#pragma unroll
          for (int t0 = 0; t0 < NT; t0 += V)
            for (int k = 0; k < 2; ++k) {
              const int left = len - t0 * LANES - k * 1024;
              if (left <= 0) break;                   // the same for all
              __syncthreads();
              if ((wv >> 1) == k) {
                f4v *to = reinterpret_cast<f4v *>(res) + (wv & 1) * 128 + lane * (V / 4);
#pragma unroll
                for (int t = t0; t < t0 + 2 * V; t += 4) {
                  const Cand p = sh[0].cand[t < t0 + V ? id0 : id1];
                  const int u = t < t0 + V ? t : t - V;
                  to[(t < t0 + V ? 0 : 256) + (u - t0) / 4] = (f4v){residual(p, u), residual(p, u + 1), residual(p, u + 2), residual(p, u + 3)};
                  __builtin_amdgcn_sched_barrier(0);
                }
              }
              __syncthreads();
              if (wv < 2) {
                const f4v *r4 = reinterpret_cast<const f4v *>(res) + wv * 256;
                const int n4 = min(256, (left + 31) / 32 * 8);      // zeros behind the last column
                f4v d[8];
                __builtin_amdgcn_s_setprio(3);
#pragma unroll
                for (int j = 0; j < 8; ++j) d[j] = r4[j];
                for (int i = 8; i <= n4; i += 8) {
#pragma unroll
                  for (int j = 0; j < 8; ++j) {
                    e = add4(e, d[j]);
                    d[j] = r4[min(i + j, 255)];
                  }
                }
                __builtin_amdgcn_s_setprio(0);
              }
            }
          if (lane == 0) sh[0].wave[wv][3] = e;
          __syncthreads();
        };
        // ---- the grid point with the least value first, then all that may be better ----
        best.e = INFINITY;
        best.id = 0x7fffffff;
        const float wl = wave_min(least);
        int wf = wave_all(least == wl ? first : 0x7fffffff, [](int x, int y) { return x < y ? x : y; });
        auto take = [&](float e, int id, const Cand &p) __attribute__((always_inline)) {
          if (e < best.e || (e == best.e && id < best.id)) {
            best.e = e;
            best.id = id;
            best.s = p.s;
            best.inv = p.inv;
            best.z = 0.f - p.a;
          }
        };
        // Points of one width often have the same step size and zero point: their errors are the same, the lower index wins
        auto same_as_best = [&](const Cand &p, int id) __attribute__((always_inline)) {
          const bool same = p.s == best.s && 0.f - p.a == best.z && best.id != 0x7fffffff;
          if (same && id < best.id) best.id = id;
          return same;
        };
        if constexpr (TW == 1) {
          auto cand_of = [&](int id) __attribute__((always_inline)) {
            const int src = id & 63, slot = id >> 6;
            Cand p = {lane_of(cd[0].s, src), lane_of(cd[0].inv, src), lane_of(cd[0].a, src), lane_of(cd[0].b, src)};
#pragma unroll
            for (int c = 1; c < CPL; ++c)
              if (slot == c) p = Cand{lane_of(cd[c].s, src), lane_of(cd[c].inv, src), lane_of(cd[c].a, src), lane_of(cd[c].b, src)};
            return p;
          };
          wf = __builtin_amdgcn_readfirstlane(wf);
          float mine[CPL];                            // errors of this lane's points that were evaluated
#pragma unroll
          for (int c = 0; c < CPL; ++c) mine[c] = INFINITY;
          if (wf != 0x7fffffff) {
            const Cand p = cand_of(wf);
            const float e = evaluate(p);
            take(e, wf, p);
#pragma unroll
            for (int c = 0; c < CPL; ++c) mine[c] = wf == lane + 64 * c ? e : mine[c];
          }
          if (any_odd) {
            // weights that are no numbers: every grid point, and if none has an error that is one, the values of point 63
            const Cand p = cand_of(63);
            best.s = p.s; best.inv = p.inv; best.z = 0.f - p.a;
          }
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            unsigned long long m = __ballot(bound[c] <= best.e * to_bins && lane + 64 * c < ncand);
            while (m) {
              const int src = __builtin_ctzll(m);
              m &= m - 1;
              const int id = src + 64 * c;
              if (id == wf || !(lane_of(bound[c], src) <= best.e * to_bins)) continue;
              const Cand p = {lane_of(cd[c].s, src), lane_of(cd[c].inv, src), lane_of(cd[c].a, src), lane_of(cd[c].b, src)};
              // Step sizes at their least value span more than the group: bounds rule nothing out, but most points are the
              // same as one before and go with it (one by one they took longer than the plain search)
              if (__builtin_bit_cast(u32, p.s) == kLeastStep) m &= ~__ballot(cd[c].s == p.s && cd[c].a == p.a);
              if (same_as_best(p, id)) continue;
              const float e = evaluate(p);
              take(e, id, p);
              mine[c] = lane == src ? e : mine[c];
            }
          }
          if (!any_odd && best.e > 0.f) {
            const float lim = best.e * close;
            int close_ones = 0;
#pragma unroll
            for (int c = 0; c < CPL; ++c)
              close_ones += __builtin_popcountll(__ballot(mine[c] <= lim && !(cd[c].s == best.s && 0.f - cd[c].a == best.z)));
            if (close_ones > 0) {
              // of all points that may be meant by one of these, also those that were taken for the same as another
#pragma unroll
              for (int c = 0; c < CPL; ++c) mine[c] = bound[c] <= lim * to_bins && lane + 64 * c < ncand && mine[c] == INFINITY ? lim : mine[c];
              best.e = INFINITY;
              best.id = 0x7fffffff;
#pragma unroll
              for (int c = 0; c < CPL; ++c) {
                unsigned long long m = __ballot(mine[c] <= lim);
                while (m) {
                  const int src = __builtin_ctzll(m);
                  m &= m - 1;
                  const Cand p = {lane_of(cd[c].s, src), lane_of(cd[c].inv, src), lane_of(cd[c].a, src), lane_of(cd[c].b, src)};
                  m &= ~__ballot(cd[c].s == p.s && cd[c].a == p.a);
                  if (!same_as_best(p, src + 64 * c)) take(in_order(p), src + 64 * c, p);
                }
              }
            }
          }
        } else {
          TeamShared &S = sh[0];
          S.cand[tid] = cd[0];
          __syncthreads();                            // the last reads of wave[][0] are done
          if (before >= 0) {                          // the same as the point before it on its diagonal: that one stands for it
            const Cand p = S.cand[before];
            if (p.s == cd[0].s && p.a == cd[0].a) bound[0] = INFINITY;
          }
          if (lane == 0) {
            S.wave[wv][0] = wl;
            S.wave[wv][1] = __builtin_bit_cast(float, wf);
          }
          __syncthreads();
          float l4 = INFINITY;
          wf = 0x7fffffff;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float l = S.wave[i][0];
            const int f = __builtin_bit_cast(int, S.wave[i][1]);
            if (l < l4 || (l == l4 && f < wf)) {
              l4 = l;
              wf = f;
            }
          }
          wf = __builtin_amdgcn_readfirstlane(wf);
          float lim = INFINITY;
          if (wf != 0x7fffffff) {
            const Cand p = S.cand[wf];
            const float e = evaluate(p);
            if (lane == 0) S.wave[wv][2] = e;
            __syncthreads();
            const float e4 = (S.wave[0][2] + S.wave[1][2]) + (S.wave[2][2] + S.wave[3][2]);
            take(e4, wf, p);
            lim = e4 * to_bins;
          } else if (any_odd) {
            const Cand p = S.cand[63];
            best.s = p.s; best.inv = p.inv; best.z = 0.f - p.a;
          }
          const unsigned long long m = __ballot(bound[0] <= lim && tid < ncand && tid != wf);
          if (lane == 0) S.alive[wv] = m;
          __syncthreads();
          int na = 0;
          for (int i = 0; i < 4; ++i) {
            unsigned long long left = uniform(S.alive[i]);
            while (left) {
              const int id = i * 64 + __builtin_ctzll(left);
              left &= left - 1;
              const float e = evaluate(S.cand[id]);
              if (lane == 0) S.part[na][wv] = e;
              ++na;
            }
          }
          __syncthreads();
          na = 0;
          for (int i = 0; i < 4; ++i) {
            unsigned long long left = uniform(S.alive[i]);
            while (left) {
              const int id = i * 64 + __builtin_ctzll(left);
              left &= left - 1;
              take((S.part[na][0] + S.part[na][1]) + (S.part[na][2] + S.part[na][3]), id, S.cand[id]);
              ++na;
            }
          }
          if (!any_odd && best.e > 0.f && na > 0) {
            // the points whose errors are close to the least, in ascending order: the first one evaluated and those listed
            const float near = best.e * close;
            float ef = INFINITY;
            if (wf != 0x7fffffff) ef = (S.wave[0][2] + S.wave[1][2]) + (S.wave[2][2] + S.wave[3][2]);
            const float bs = best.s, bz = best.z;
            int others = 0, count = 0;
            bool more = false;                        // than four of them
            int ids[4] = {0, 0, 0, 0};
            for (int pass = 0; pass < 2; ++pass) {    // looks for one beside the best, then ranks them, four at a time
              int k = 0;
              bool first_due = ef <= near;
              if (pass == 1) {
                if (more) count = 0;
                best.e = INFINITY;
                best.id = 0x7fffffff;
              }
              auto rank = [&]() __attribute__((always_inline)) {
                for (int c = 0; c < count; c += 2) {
                  const int id0 = c == 0 ? ids[0] : ids[2], id1 = c == 0 ? (count > 1 ? ids[1] : id0) : (count > 3 ? ids[3] : id0);
                  in_order2(id0, id1);
                  take(S.wave[0][3], id0, S.cand[id0]);
                  take(S.wave[1][3], id1, S.cand[id1]);
                  __syncthreads();                    // read before the next two sums are written
                }
                count = 0;
              };
              // at the least step size the points of one lower end are the same: the first of a run stands for it
              float last_s = 0.f, last_a = 0.f;
              auto due = [&](int id) __attribute__((always_inline)) {
                const Cand p = S.cand[id];
                if (p.s == last_s && p.a == last_a) return;
                last_s = p.s;
                last_a = p.a;
                others += p.s == bs && 0.f - p.a == bz ? 0 : 1;
#pragma unroll
                for (int c = 0; c < 4; ++c) ids[c] = c == count ? id : ids[c];
                ++count;
              };
              for (int i = 0; i < 4 && (pass == 0 || more); ++i) {
                unsigned long long left = uniform(S.alive[i]);
                while (left) {
                  const int id = i * 64 + __builtin_ctzll(left);
                  const bool close_one = (S.part[k][0] + S.part[k][1]) + (S.part[k][2] + S.part[k][3]) <= near;
                  const bool first_now = first_due && wf < id;
                  if (!first_now) {
                    left &= left - 1;
                    ++k;
                  }
                  first_due = first_due && !first_now;
                  if (first_now || close_one) due(first_now ? wf : id);
                  if (count == 4) {
                    if (pass == 1) rank();
                    more = true;
                    count = 0;
                  }
                }
              }
              if (first_due && (pass == 0 || more)) due(wf);
              if (others == 0) break;
              if (pass == 1 && count > 0) rank();
            }
          }
        }
      }
    }
    team_barrier();                                // the histogram is cleared for the next group
    if (BITS > 0 && left) {
      if (lane == 0) a.scale[(size_t)row * a.n_groups + gi] = kLeft;
      row = nrow;
      gi = ngi;
      continue;
    }
    if (TW == 1 || wv == 0) store_choice(a, row, gi, best, lane);
    uint8_t *crow = a.codes + (size_t)row * a.d_in + c0;
    typedef uint8_t bv __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int t = 0; t < NT; t += V) {
      const int c = T::column(t, tl);
      bv q;
      if constexpr (V >= 4) {
        typedef u32 wv_t __attribute__((ext_vector_type(V / 4)));
        wv_t words;
#pragma unroll
        for (int e = 0; e < V; e += 4) {
          u32 w = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) w |= (u32)code_of(cur[t + e + i], best, a.qmax) << (8 * i);
          // four bits of `kept` to four bytes
          const u32 in = (((nothing ? 0u : (u32)(kept >> ((t + e) & 32))) >> ((t + e) & 31)) & 15u) * 0x00204081u & 0x01010101u;
          words[e / 4] = w & ((in << 8) - in);
        }
        q = __builtin_bit_cast(bv, words);
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) q[e] = (nothing || !((kept >> (t + e)) & 1u)) ? (uint8_t)0 : code_of(cur[t + e], best, a.qmax);
      }
      if (a.vec) {
        if (c < len) *reinterpret_cast<bv *>(crow + c) = q;
      } else {
        const int l = seldom(tl);
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (T::column(t + e, l) < len) crow[T::column(t + e, l)] = q[e];
      }
    }
    row = nrow;
    gi = ngi;
  }
}

// ---------------------------------------------------------------------------
// plain search of long rows
// ---------------------------------------------------------------------------
// The grid points of this lane for the range [lo, hi], errors cleared.
template <int CPL>
__device__ __forceinline__ void make_cands(float lo, float hi, const float (&fa)[CPL], const float (&fb)[CPL],
                                           float qmax, Cand (&cd)[CPL], float (&e)[CPL]) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    cd[c] = candidate<true>(lo, hi, fa[c], fb[c], qmax, 0.f);
    e[c] = 0.f;
  }
}

// Adds the errors of list[0 .. cnt) to every grid point of this lane.
template <int CPL>
__device__ __forceinline__ void accumulate_list(const float *list, int cnt, const Cand (&cd)[CPL], float (&e)[CPL]) {
  const f4v *l4 = reinterpret_cast<const f4v *>(list);
  int i = 0;
  f4v nxt = l4[0];                                 // one address for the wave: a broadcast
  for (; i + 4 <= cnt; i += 4) {
    const f4v v = nxt;
    nxt = l4[(i >> 2) + 1];                        // one step ahead (the list has four spare entries)
    accumulate<CPL>(cd, e, v[0]);
    accumulate<CPL>(cd, e, v[1]);
    accumulate<CPL>(cd, e, v[2]);
    accumulate<CPL>(cd, e, v[3]);
  }
  for (; i < cnt; ++i) accumulate<CPL>(cd, e, list[i]);
}

// Ranks this lane's grid points, then the wave's; equal errors go to the lower index.  The
// winner's step size and zero point are read from the lane that holds them.
template <int CPL>
__device__ __forceinline__ Best pick(const Cand (&cd)[CPL], const float (&e)[CPL], int ncand, int lane) {
  float eb = INFINITY;
  int ib = 0x7fffffff;
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int id = lane + 64 * c;
    if (id < ncand && (e[c] < eb || (e[c] == eb && id < ib))) {
      eb = e[c];
      ib = id;
    }
  }
  const float e_min = wave_all(eb, [](float x, float y) { return x < y ? x : y; });
  ib = wave_all(eb == e_min ? ib : 0x7fffffff, [](int x, int y) { return x < y ? x : y; });
  ib = __builtin_amdgcn_readfirstlane(ib);
  const int slot = ib >> 6, src = ib & 63;
  auto from_lane = [&](float v) __attribute__((always_inline)) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
  };
  Best b;
  b.s = from_lane(cd[0].s);
  b.inv = from_lane(cd[0].inv);
  float neg_z = from_lane(cd[0].a);
#pragma unroll
  for (int c = 1; c < CPL; ++c) {                  // slot is the same for the whole wave
    const float s = from_lane(cd[c].s), inv = from_lane(cd[c].inv), na = from_lane(cd[c].a);
    b.s = slot == c ? s : b.s;
    b.inv = slot == c ? inv : b.inv;
    neg_z = slot == c ? na : neg_z;
  }
  b.z = 0.f - neg_z;
  b.e = e_min;
  b.id = ib;
  return b;
}

// Groups of more than 16384 columns, which four waves do not hold in registers: one wave per group, moved through
// LDS kChunk columns at a time, three passes over the row (range, errors, codes).
template <int CPL>
__global__ __launch_bounds__(kWaves * 64) void owq_search_kernel(const SearchArgs a) {
  __shared__ __attribute__((aligned(16))) float lists[kWaves][kChunk + 4];   // + 4: read one step ahead
  extern __shared__ u32 mask[];                    // bit c = column c is weak; (d_in + 31) / 32 words
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  float *list = lists[wv];
  // every thread of the workgroup passes these two barriers before anything may leave
  for (int i = threadIdx.x; i < (a.d_in + 31) >> 5; i += kWaves * 64) mask[i] = 0u;
  __syncthreads();
  for (int p = threadIdx.x; p < a.k; p += kWaves * 64) {
    const u32 c = (u32)a.weak_idx[p];
    if (c < (u32)a.d_in) atomicOr(&mask[c >> 5], 1u << (c & 31));
  }
  __syncthreads();
  const int ncand = a.n_lo * a.n_hi;
  // the cut fractions of this lane's grid points do not depend on the group
  float fa[CPL], fb[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int id = lane + 64 * c;
    const int i = id / a.n_hi, j = id - i * a.n_hi;
    fa[c] = cut_fraction(a.shrink, i < a.n_lo ? i : 0, a.n_lo);
    fb[c] = cut_fraction(a.shrink, j, a.n_hi);
  }
  const int u0 = (blockIdx.x * kWaves + wv) * a.units_per_wave;
  const int n_units = a.units - u0 < a.units_per_wave ? a.units - u0 : a.units_per_wave;   // same for the wave
  if (n_units <= 0) return;
  int row = u0 / a.n_groups, gi = u0 - row * a.n_groups;
  const Best none = {1.f, 1.f, 0.f, 0.f, 0};

  for (int uu = 0; uu < n_units; ++uu) {
    const int c0 = gi * a.g;
    const int len = a.d_in - c0 < a.g ? a.d_in - c0 : a.g;
    const _Float16 *wrow = a.w + (size_t)row * a.d_in;
    // least and greatest non-weak weight
    float lo = INFINITY, hi = -INFINITY;
    int kept = 0;
    for (int o = 0; o < len; o += kChunk) {
      const int cnt = stage(wrow, c0 + o, len - o < kChunk ? len - o : kChunk, list, mask, lane);
      kept += cnt;
      for (int e = lane; e < cnt; e += 64) {
        const float v = list[e];
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
      }
      wave_lds_fence();
    }
    lo = wave_all(lo, [](float x, float y) { return x < y ? x : y; });
    hi = wave_all(hi, [](float x, float y) { return x > y ? x : y; });
    const bool nothing = degenerate(lo, hi, kept);
    Best best = none;
    if (!nothing) {
      Cand cd[CPL];
      float e[CPL];
      make_cands<CPL>(lo, hi, fa, fb, a.qmax, cd, e);
      for (int o = 0; o < len; o += kChunk) {
        const int cnt = stage(wrow, c0 + o, len - o < kChunk ? len - o : kChunk, list, mask, lane);
        accumulate_list<CPL>(list, cnt, cd, e);
        wave_lds_fence();                        // the list is rewritten by the next pass
      }
      best = pick<CPL>(cd, e, ncand, lane);
    }
    store_choice(a, row, gi, best, lane);
    // the codes of the group under the chosen step size and zero point; 0 at weak columns
    uint8_t *crow = a.codes + (size_t)row * a.d_in;
    for (int c = c0 + lane; c < c0 + len; c += 64)
      crow[c] = (nothing || is_weak(mask, c)) ? (uint8_t)0 : code_of((float)wrow[c], best, a.qmax);
    if (++gi == a.n_groups) {
      gi = 0;
      ++row;
    }
  }
}

typedef void (*search_fn)(const SearchArgs);
template <int POINTS, int BITS>
search_fn pick_bounds_wave(int g) {
  if (g <= 128) return owq_search_bounds<1, 2, POINTS, BITS>;
  if (g <= 256) return owq_search_bounds<1, 4, POINTS, BITS>;
  if (g <= 512) return owq_search_bounds<1, 8, POINTS, BITS>;
  return owq_search_bounds<1, 16, POINTS, BITS>;
}
search_fn pick_bounds(int g, int ncand) {
  if (g <= 1024)
    return ncand <= 64 ? pick_bounds_wave<1, 0>(g) : ncand <= 128 ? pick_bounds_wave<2, 0>(g) : ncand <= 192 ? pick_bounds_wave<3, 0>(g) : pick_bounds_wave<4, 0>(g);
  if (g <= 2048) return owq_search_bounds<4, 8, 1, 0>;
  if (g <= 4096) return owq_search_bounds<4, 16, 1, 0>;
  if (g <= 6144) return owq_search_bounds<4, 24, 1, 0>;
  if (g <= 8192) return owq_search_bounds<4, 32, 1, 0>;
  if (g <= 12288) return owq_search_bounds<4, 48, 1, 0>;
  return owq_search_bounds<4, 64, 1, 0>;
}
constexpr int kBoundsMax = 16384;    // columns of the longest group four waves keep in registers

}  // namespace
}  // namespace owq

extern "C" owq_status_t owq_search_config(const owq_search_desc_t *d, const uint16_t *w, const int32_t *weak_idx,
                                          uint16_t *scale, uint16_t *zero, uint8_t *codes, float *err,
                                          int32_t *choice, void *stream) {
  using namespace owq;
  if (!d || !w || !scale || !zero || !codes) return OWQ_ERR_NULL;
  if (d->d_out < 1 || d->d_in < 1) return OWQ_ERR_SHAPE;
  if (d->bits != 3 && d->bits != 4) return OWQ_ERR_BITS;
  if (d->group_size < 0 || d->group_size % 128 != 0) return OWQ_ERR_GROUP;
  if (d->k < 0 || d->k > d->d_in) return OWQ_ERR_INDEX;
  if (d->k > 0 && !weak_idx) return OWQ_ERR_NULL;
  if (d->n_lo < 1 || d->n_lo > 16 || d->n_hi < 1 || d->n_hi > 16) return OWQ_ERR_SHAPE;
  if (!(d->shrink >= 0.f && d->shrink < 0.5f)) return OWQ_ERR_SHAPE;
  const int g = d->group_size == 0 || d->group_size > d->d_in ? d->d_in : d->group_size;
  const long long n_groups = (d->d_in + (long long)g - 1) / g;
  const long long units = n_groups * d->d_out;
  if (units > 0x7fffffffLL) return OWQ_ERR_SHAPE;
  const size_t mask_bytes = (size_t)((d->d_in + 31) / 32) * 4;
  if (mask_bytes > (size_t)kMaskBytesMax) return OWQ_ERR_UNSUPPORTED;
  SearchArgs a;
  a.w = reinterpret_cast<const _Float16 *>(w);
  a.weak_idx = weak_idx;
  a.scale = scale;
  a.zero = zero;
  a.codes = codes;
  a.err = err;
  a.choice = choice;
  a.d_in = d->d_in;
  a.g = g;
  a.n_groups = (int)n_groups;
  a.k = d->k;
  a.n_lo = d->n_lo;
  a.n_hi = d->n_hi;
  a.units = (int)units;
  // several groups per team once there are enough teams to fill the chip many times over: the
  // per-lane grid set-up and the weak mask are then paid once per team
  const bool bounds = g <= kBoundsMax;
  const int team_waves = bounds && g > 1024 ? 4 : 1;
  // (four waves: two rows where there are 16384, 120 -> 115 us on rows of 4096; of 5120 rows, two each take 81 us and one 77)
  const long long upw = units / (team_waves == 4 ? 8192 : 32768);
  a.units_per_wave = (int)(upw < 1 ? 1 : (upw > 16 ? 16 : upw));
  a.qmax = (float)((1 << d->bits) - 1);
  a.shrink = d->shrink;
  const int run = g <= 128 ? 2 : g <= 256 ? 4 : 8;   // columns a lane of owq_search_bounds reads at once
  a.vec = d->d_in % run == 0 && reinterpret_cast<uintptr_t>(w) % (2 * run) == 0 && reinterpret_cast<uintptr_t>(codes) % run == 0;
  const long long teams = (units + a.units_per_wave - 1) / a.units_per_wave;
  const int per_wg = kWaves / team_waves;
  const dim3 grid((unsigned)((teams + per_wg - 1) / per_wg)), block(kWaves * 64);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int ncand = d->n_lo * d->n_hi;
  // By diagonals: as many points at either end, so that the cuts of a diagonal add up to one sum; more than two points a lane
  // (with two the general grid's kernel takes as few lookups); steps of a diagonal's width that are several steps of binary16,
  // so that no two diagonals have the same step size; and weights enough that what it saves (0.6 us per 2^17 weights or more) is
  // more than the second launch costs (5 us).
  bool diagonals = bounds && g <= 1024 && d->n_lo == d->n_hi && ncand > 128 && d->shrink * 256.f >= (float)(d->n_lo - 1) &&
                   (long long)d->d_out * d->d_in >= (4 << 20) && units >= 16384;
  // And no run of zero points longer than a lane takes: from 0.45 on at 4 bits (0.46 at 3) some groups have longer ones, and a
  // launch that finds any takes 10 us more (4096 x 4096, 4-bit, 12 x 12 points of 0.45, groups of 512: 64 us, weights spread evenly 83;
  // the general grid's kernel 57 and 54; groups of 128 134 and 152, so 135 and 132).
  const float cut = d->shrink / (float)(d->n_lo - 1);
  for (int c = 0; diagonals && c <= 2 * (d->n_lo - 1); ++c) {
    const int points = (c < d->n_lo ? c : 2 * (d->n_lo - 1) - c) + 1;
    diagonals = (float)((points - 1) / 2) * cut * a.qmax <= (float)(zero_points(d->bits) - 1) * (1.f - cut * (float)c);
  }
  if (diagonals) {
    hipLaunchKernelGGL((d->bits == 3 ? pick_bounds_wave<4, 3>(g) : pick_bounds_wave<4, 4>(g)), grid, block, mask_bytes, st, a);
    if (hipGetLastError() != hipSuccess) return OWQ_ERR_HIP;
    const long long left = units / 8192;
    a.units_per_wave = (int)(left < 1 ? 1 : left > 64 ? 64 : left);
    const long long waves = (units + a.units_per_wave - 1) / a.units_per_wave;
    hipLaunchKernelGGL((pick_bounds_wave<4, -1>(g)), dim3((unsigned)((waves + kWaves - 1) / kWaves)), block, mask_bytes, st, a);
  } else {
    const search_fn fn = bounds ? pick_bounds(g, ncand)
                         : ncand <= 64 ? owq_search_kernel<1> : ncand <= 128 ? owq_search_kernel<2> : ncand <= 192 ? owq_search_kernel<3> : owq_search_kernel<4>;
    hipLaunchKernelGGL(fn, grid, block, mask_bytes, st, a);
  }
  return hipGetLastError() == hipSuccess ? OWQ_OK : OWQ_ERR_HIP;
}
