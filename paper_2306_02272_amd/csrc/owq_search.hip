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
// and then those whose bound, less a bound on its own rounding, does not exceed the least error found: five of 256
// on groups of 128, one or two on long rows.  These evaluations take the same binary32 decisions per weight as the
// plain search and share their sums among the lanes; points whose sums come out too close to tell are summed again in
// the order of the columns, so that the choice is that of the plain search.
// 16384 x 4096, 3-bit, groups of 128, 16 x 16 points: 1780 -> 620 us (bound by vector instructions, 815 per group by the
// counter where the plain search spent 3000); 5120 x 5120, 4-bit, one scale per row: 717 -> 127-138 us from box to box (of
// which 30 are the few rows with points to tell apart).
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

template <int TW, int NT, int POINTS>
__global__ __launch_bounds__(256) void owq_search_bounds(const SearchArgs a) {
  using T = Team<TW, NT, POINTS>;
  constexpr int V = T::V, LANES = T::LANES, F = T::F, CPL = T::CPL, TEAMS = 4 / TW;
  __shared__ __attribute__((aligned(16))) unsigned long long hist[TEAMS][F + 2];
  __shared__ TeamShared sh[1];                     // four waves only
  extern __shared__ u32 mask[];                    // bit c = column c is weak; (d_in + 31) / 32 words
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int tl = TW == 4 ? tid : lane;             // lane within the team
  unsigned long long *bins = hist[TW == 4 ? 0 : wv];
  for (int i = tid; i < (a.d_in + 31) >> 5; i += 256) mask[i] = 0u;
  __syncthreads();
  for (int p = tid; p < a.k; p += 256) {
    const u32 c = (u32)a.weak_idx[p];
    if (c < (u32)a.d_in) atomicOr(&mask[c >> 5], 1u << (c & 31));
  }
  __syncthreads();
  const int ncand = a.n_lo * a.n_hi;
  float fa[CPL], fb[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int id = tl + LANES * c;
    const int i = id / a.n_hi, j = id - i * a.n_hi;
    fa[c] = cut_fraction(a.shrink, i < a.n_lo ? i : 0, a.n_lo);
    fb[c] = cut_fraction(a.shrink, j, a.n_hi);
  }
  const int team = TW == 4 ? (int)blockIdx.x : (int)blockIdx.x * 4 + wv;
  const int u0 = team * a.units_per_wave;
  const int n_units = a.units - u0 < a.units_per_wave ? a.units - u0 : a.units_per_wave;   // same for the team
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
#pragma unroll
    for (int t = 0; t < NT; t += V) {
      const int c = T::column(t, tl);
      if (a.vec) {                                 // rows on the grid of V elements, len a multiple of V
        const hv v = *reinterpret_cast<const hv *>(src + (c < len ? c : len - V));
#pragma unroll
        for (int e = 0; e < V; ++e) dst[t + e] = v[e];
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) dst[t + e] = src[c + e < len ? c + e : len - 1];
      }
    }
  };
  // a wave fetches its next group while it searches one; with four waves to a row other workgroups fill the wait
  constexpr bool kAhead = TW == 1;
  float cur[NT];
  _Float16 nxt[NT];
  fetch(nxt, row, gi);
  for (int uu = 0; uu < n_units; ++uu) {
    const int c0 = gi * a.g;
    const int len = a.d_in - c0 < a.g ? a.d_in - c0 : a.g;
    int nrow = row, ngi = gi + 1;
    if (ngi == a.n_groups) {
      ngi = 0;
      ++nrow;
    }
    if (!kAhead && uu > 0) fetch(nxt, row, gi);
#pragma unroll
    for (int t = 0; t < NT; ++t) cur[t] = (float)nxt[t];
    if (kAhead && uu + 1 < n_units) fetch(nxt, nrow, ngi);
    // ---- range; an empty histogram ----
    unsigned long long kept = 0;                   // bit t: weight t of this lane takes part
    float lo = INFINITY, hi = -INFINITY;
    bool odd = false;                              // a weight that is no number
#pragma unroll
    for (int t = 0; t < NT; t += V) {
      const int c = T::column(t, tl);
      u32 m = 0u;
      if (c < len) {
        m = ~(mask[(c0 + c) >> 5] >> ((c0 + c) & 31)) & ((1u << V) - 1u);
        if (len - c < V) m &= (1u << (len - c)) - 1u;
      }
      kept |= (unsigned long long)m << t;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const float v = cur[t + e];
        const bool in = (m >> e) & 1u;
        odd |= in && !(__builtin_fabsf(v) < INFINITY);
        lo = __builtin_fminf(lo, in ? v : INFINITY);      // ignores what is no number
        hi = __builtin_fmaxf(hi, in ? v : -INFINITY);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) bins[tl * 4 + i] = 0ull;
    lo = wave_all(lo, [](float x, float y) { return __builtin_fminf(x, y); });
    hi = wave_all(hi, [](float x, float y) { return __builtin_fmaxf(x, y); });
    int cnt = 0;                                   // kept weights of the wave
#pragma unroll
    for (int t = 0; t < NT; ++t) cnt += __builtin_popcountll(__ballot((kept >> t) & 1u));
    bool any_odd = __ballot(odd) != 0ull;
    if constexpr (TW == 4) {
      if (lane == 0) {
        sh[0].wave[wv][0] = lo;
        sh[0].wave[wv][1] = hi;
        sh[0].wave[wv][2] = (float)cnt;
        sh[0].wave[wv][3] = any_odd ? 1.f : 0.f;
      }
      __syncthreads();
      cnt = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float l = sh[0].wave[i][0], h = sh[0].wave[i][1];
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
        cnt += (int)sh[0].wave[i][2];
        any_odd |= sh[0].wave[i][3] != 0.f;
      }
    } else {
      wave_lds_fence();
    }
    const bool nothing = degenerate(lo, hi, cnt);
    Best best = {1.f, 1.f, 0.f, 0.f, 0};
    if (!nothing) {
      Cand cd[CPL];
      float bound[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        cd[c] = candidate<false>(lo, hi, fa[c], fb[c], a.qmax, 1.f / a.qmax);
        bound[c] = -INFINITY;
      }
      if (any_odd) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) cd[c] = candidate<true>(lo, hi, fa[c], fb[c], a.qmax, 0.f);
      }
      // error of grid point (s, inv, za, zb) over this lane's weights, over the wave
      auto evaluate = [&](const Cand &p) __attribute__((always_inline)) {
        float e = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float v = cur[t];
          const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(v * p.inv), p.a, p.b);   // q - z
          float d = __builtin_fmaf(-p.s, q, v);
          d = (kept >> t) & 1u ? d : 0.f;
          e = __builtin_fmaf(d, d, e);
        }
        return wave_sum(e);
      };
      const float idelta = (float)F / (hi - lo);
      float least = INFINITY;                      // least value (not bound) from the table, and its grid point
      int first = 0x7fffffff;
      if (!any_odd) {
        // ---- histogram: count in the upper half, sum of the offsets inside the bin (in 2^-16 bins) in the lower ----
        float s2 = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float u = (cur[t] - lo) * idelta;
          int b = (int)u;
          b = b < 0 ? 0 : (b > F - 1 ? F - 1 : b);
          const float f = __builtin_fminf(__builtin_fmaxf(u - (float)b, 0.f), 1.f);
          const float uc = u - (float)(F / 2);
          if ((kept >> t) & 1u) {
            atomicAdd(&bins[b], (1ull << 32) | (unsigned long long)(u32)(f * 65536.f + 0.5f));
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
        float dg[4], d4 = 0.f;
        int below = incl - n4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int n = (int)(h[i] >> 32);
          dg[i] = -(float)below - ((float)n - (float)(u32)h[i] * 0x1p-16f);
          below += n;
          d4 += dg[i];
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
        // ---- bounds ----
        // What rounding can do to a value: eight operations on terms of at most `mag`, and positions (midpoints, levels)
        // that are off by `eps` bins, each seen by all weights
        const float far = __builtin_fmaxf(__builtin_fabsf(lo), __builtin_fabsf(hi)) * idelta, half = (float)(F / 2);
        const float mag = 2.f * (s2 + half * (half * n + 2.f * __builtin_fabsf(s1)));
        const float eps = 3.f * (float)F + 2.f * far;
        const float slack = 0x1p-24f * (8.f * mag + 4.f * n * (float)F * eps);
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
      // The error of a grid point as one sum in the order of the columns, which is what ranks points whose errors agree to
      // the rounding of such sums: the residuals go through LDS (where the bins were), the sum runs on every lane.
      auto residual = [&](const Cand &p, int t) __attribute__((always_inline)) {
        const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(cur[t] * p.inv), p.a, p.b);
        return (kept >> t) & 1u ? __builtin_fmaf(-p.s, q, cur[t]) : 0.f;
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
          for (int i = 0; i < n4; ++i) e = add4(e, reinterpret_cast<const f4v *>(res)[i]);
        }
        return e;
      };
      // Four waves: wave c sums point c of up to four; the residuals come 512 columns (one wave's run of them) at a time, 32
      // in registers while the next 32 come from LDS.  One point after the other, a chain of LDS reads each, took 87 us
      // per point on a row of 5120 columns.
      auto in_order4 = [&](const int (&ids)[4], int count) __attribute__((always_inline)) {
        float e = 0.f;
#pragma unroll
        for (int t0 = 0; t0 < NT; t0 += V)
          for (int k = 0; k < 4; ++k) {
            const int left = len - t0 * LANES - k * 512;
            if (left <= 0) break;                   // the same for all
            __syncthreads();
            if (wv == k) {
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (c < count) {
                  const Cand p = sh[0].cand[ids[c]];
#pragma unroll
                  for (int t = t0; t < t0 + V; ++t) res[c * 512 + lane * V + t - t0] = residual(p, t);
                }
            }
            __syncthreads();
            if (wv < count) {
              const f4v *r4 = reinterpret_cast<const f4v *>(res) + wv * 128;
              const int n4 = min(128, (left + 31) / 32 * 8);
              f4v d[8], nx[8];
#pragma unroll
              for (int j = 0; j < 8; ++j) d[j] = r4[j];
              for (int i = 0; i < n4; i += 8) {
#pragma unroll
                for (int j = 0; j < 8; ++j) nx[j] = r4[(i + 8 < 128 ? i + 8 : i) + j];
#pragma unroll
                for (int j = 0; j < 8; ++j) e = add4(e, d[j]);
#pragma unroll
                for (int j = 0; j < 8; ++j) d[j] = nx[j];
              }
            }
          }
        if (lane == 0) sh[0].wave[wv][3] = e;
        __syncthreads();
      };
      // errors this close may change places: four deviations of the rounding of two sums of cnt terms (0.3 sqrt(cnt / 3) units in
      // the 24th place each)
      const float close = 1.f + 0x1p-24f * (__builtin_sqrtf((float)cnt) + 8.f);
      // ---- the grid point with the least value first, then all that may be better ----
      const float to_bins = any_odd ? 1.f : idelta * idelta * (1.f + 0x1p-12f);
      best.e = INFINITY;
      best.id = 0x7fffffff;
      const float wl = wave_all(least, [](float x, float y) { return __builtin_fminf(x, y); });
      int wf = wave_all(least == wl ? first : 0x7fffffff, [](int x, int y) { return x < y ? x : y; });
      auto lane_of = [&](float v, int src) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
      };
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
          int found = 0, count = 0;
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
              in_order4(ids, count);
              for (int c = 0; c < count; ++c) {
                const int id = c == 0 ? ids[0] : c == 1 ? ids[1] : c == 2 ? ids[2] : ids[3];
                take(S.wave[c][3], id, S.cand[id]);
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
              found += p.s == bs && 0.f - p.a == bz ? 0 : 1;
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
            if (found == 0) break;
            if (pass == 1 && count > 0) rank();
          }
        }
      }
    }
    team_barrier();                                // the histogram is cleared for the next group
    if (TW == 1 || wv == 0) store_choice(a, row, gi, best, lane);
    uint8_t *crow = a.codes + (size_t)row * a.d_in + c0;
    typedef uint8_t bv __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int t = 0; t < NT; t += V) {
      const int c = T::column(t, tl);
      bv q;
#pragma unroll
      for (int e = 0; e < V; ++e)
        q[e] = (nothing || !((kept >> (t + e)) & 1u)) ? (uint8_t)0 : code_of(cur[t + e], best, a.qmax);
      if (a.vec) {
        if (c < len) *reinterpret_cast<bv *>(crow + c) = q;
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (c + e < len) crow[c + e] = q[e];
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
template <int POINTS>
search_fn pick_bounds_wave(int g) {
  if (g <= 128) return owq_search_bounds<1, 2, POINTS>;
  if (g <= 256) return owq_search_bounds<1, 4, POINTS>;
  if (g <= 512) return owq_search_bounds<1, 8, POINTS>;
  return owq_search_bounds<1, 16, POINTS>;
}
search_fn pick_bounds(int g, int ncand) {
  if (g <= 1024)
    return ncand <= 64 ? pick_bounds_wave<1>(g) : ncand <= 128 ? pick_bounds_wave<2>(g) : ncand <= 192 ? pick_bounds_wave<3>(g) : pick_bounds_wave<4>(g);
  if (g <= 2048) return owq_search_bounds<4, 8, 1>;
  if (g <= 4096) return owq_search_bounds<4, 16, 1>;
  if (g <= 6144) return owq_search_bounds<4, 24, 1>;
  if (g <= 8192) return owq_search_bounds<4, 32, 1>;
  if (g <= 12288) return owq_search_bounds<4, 48, 1>;
  return owq_search_bounds<4, 64, 1>;
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
  const long long upw = units / (team_waves == 4 ? 2048 : 32768);
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
  const search_fn fn = bounds ? pick_bounds(g, ncand)
                       : ncand <= 64 ? owq_search_kernel<1> : ncand <= 128 ? owq_search_kernel<2> : ncand <= 192 ? owq_search_kernel<3> : owq_search_kernel<4>;
  hipLaunchKernelGGL(fn, grid, block, mask_bytes, st, a);
  return hipGetLastError() == hipSuccess ? OWQ_OK : OWQ_ERR_HIP;
}
