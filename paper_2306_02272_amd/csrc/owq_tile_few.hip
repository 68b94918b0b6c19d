// Tile layout, 32 tokens or fewer, one launch: every workgroup owns its rows for all columns.
//
//     y[n,i] = sum_{j not weak} s_ig (q_ij - z_ig) x[n,j]  +  sum_t Ww_it x[n, idx_t]
//
// With few tokens a call is bound by the stream of codes and by latency.  The kernel of owq_tile_small.hip spreads a
// row tile's columns over several workgroups, stages a range of activations before anything else and needs a second
// launch for the sums (4.5 us, and a gap, of 16 on a 5120 x 5120 layer at 16 tokens).  Here a workgroup takes one or
// two row tiles of 32 rows and ALL columns; its waves (eight, or four above 16 tokens) take a run of 128-column blocks
// each, and add their results through LDS at the end.  A wave's blocks come by direct loads to LDS, codes and
// activations alike, two blocks ahead, into a ring of its own: no registers are held by loads in flight, the
// waits are exact, and there is no barrier between the start and the sums.
//
//   x       rows of 256 bytes per token and block, 16-byte units exchanged by the low bits of the token (operand reads
//           free of bank conflicts); the values at weak columns are moved to the operand of the weak product and
//           overwritten with zeros by the wave that fetched them;
//   codes   A operand q - z, exactly (see a_exact), per 128-column block from zero, then one fused multiply-add per
//           value with the step size; zero points that are no integers of at most 1024 take a side path;
//   weak    a few k-steps at the end, dealt out to the waves.
// No atomics; sums in a fixed order.
#include <hip/hip_runtime.h>

#include "owq_internal.h"
#include "owq_tile_device.h"

namespace owq {
namespace {

constexpr int kFewKp = 512;           // most (padded) weak columns: the gathered activations lie in LDS
constexpr int kFewLds = 160 * 1024;

struct FewArgs {
  const unsigned char *codes;
  const u32 *sz;               // [n_groups][d_out_pad]: fp16 scale | fp16 zero << 16
  const int *weak_idx;         // [kp], padding -1
  const u32x4 *weak_w;         // [d_out_pad][kp/8] units
  const _Float16 *x;           // [ntok][d_in], 16-byte aligned rows
  _Float16 *y;                 // [ntok][d_out]
  int d_in, d_out, d_out_pad, n_rt, ntok, nbp, nblk, n_groups, bpg, k, kp;
  int lg_tok;                  // tokens are padded to 1 << lg_tok (4 to 32) in LDS
  // LDS byte offsets: scales [row tile][group][32 rows], gathered activations [token][kp] and the dwords they are picked
  // from, weak indices
  int off_sz, off_xw, off_xd, off_idx;
};

// A dword per lane to LDS at lds + 4 * lane.
__device__ __forceinline__ void dword_to_lds(const void *sbase, u32 voff, u32 lds) {
  u32 m0;      // see load_to_lds
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, %3" : "=&{m0}"(m0) : "s"(lds), "v"(voff), "s"(sbase) : "memory");
}

// As load_to_lds, N times 1 KB further on both sides: sbase + voff + 1024 i to lds + 1024 i + 16 lane, i < N <= 4.  One
// write of the LDS base serves all of them.
template <int N>
__device__ __forceinline__ void loads_to_lds(const void *sbase, const u32 *voff, u32 lds) {
  static_assert(N == 1 || N == 2 || N == 4, "the offset field holds 3072");
  u32 m0;      // see load_to_lds
  if constexpr (N == 1)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" : "=&{m0}"(m0) : "s"(lds), "v"(voff[0]), "s"(sbase) : "memory");
  else if constexpr (N == 2)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %4\n\tglobal_load_lds_dwordx4 %3, %4 offset:1024"
                 : "=&{m0}"(m0) : "s"(lds), "v"(voff[0]), "v"(voff[1]), "s"(sbase) : "memory");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %6\n\tglobal_load_lds_dwordx4 %3, %6 offset:1024\n\t"
                 "global_load_lds_dwordx4 %4, %6 offset:2048\n\tglobal_load_lds_dwordx4 %5, %6 offset:3072"
                 : "=&{m0}"(m0) : "s"(lds), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(sbase) : "memory");
}

template <int BITS, int RT, int S>
struct FewSteps {
  static __device__ __forceinline__ void run(const u32 (*wd)[8], const unsigned char *xb, u32 xsw, const Magic &M, const u32 (*nb)[8],
                                             f16_t *acc, const f16_t &zero) {
    const h8_t b = *reinterpret_cast<const h8_t *>(xb + (xsw ^ (S << 5)));
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = mma(a_exact<BITS, S>(wd[t], M, nb[t]), b, S == 0 ? zero : acc[t]);
    FewSteps<BITS, RT, S + 1>::run(wd, xb, xsw, M, nb, acc, zero);
  }
};
template <int BITS, int RT>
struct FewSteps<BITS, RT, 8> {
  static __device__ __forceinline__ void run(const u32 (*)[8], const unsigned char *, u32, const Magic &, const u32 (*)[8], f16_t *,
                                             const f16_t &) {}
};

constexpr int kFewDepth = 2;          // blocks in flight per wave; three and four measured the same

// grid: groups of RT row tiles; 4 or 8 waves; 4 NX tokens or fewer.  What bounds it is the issue of instructions, about
// 230 per block and row tile (unpack 72, matrix 8, scaling 24, LDS reads 14, weak columns, loads): the loads are made of
// as few of them as possible.
template <int BITS, int RT, int NX>
__global__ __launch_bounds__(512, 2) void owq_tile_few(const FewArgs a) {
  extern __shared__ u32x4 lds_units[];
  unsigned char *lds = reinterpret_cast<unsigned char *>(lds_units);
  const u32 ldsb = lds_address(lds);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), W = blockDim.x >> 6;
  const int n32 = lane & 31, kg = lane >> 5;
  constexpr int np = 4 * NX, D = kFewDepth, stage = np * 256 + RT * 2048, kPer = NX + 2 * RT;   // kPer: loads of a block
  const int ring = w * D * stage;
  const int rg = blockIdx.x;
  const int lg_w = W == 8 ? 3 : 2, b0 = (w * a.nblk) >> lg_w, b1 = ((w + 1) * a.nblk) >> lg_w;
  constexpr int CH = BITS == 3 ? 3 : 4;

  // ---- fetch: token rows 4i .. 4i+3 of a block per load (a quarter wave per row), two chunks of codes per row tile ----
  // (xoff: less the 1024 i that the load adds, and 8192 to stay above zero)
  u32 xoff[NX];
  int xoct[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int n = 4 * i + (lane >> 4), gn = n < a.ntok ? n : a.ntok - 1;      // tokens past the end: any row
    xoct[i] = (lane & 15) ^ (n & 15);
    xoff[i] = (u32)gn * (u32)(a.d_in * 2) + (u32)xoct[i] * 16u + 8192u - 1024u * (u32)(i & 3);
  }
  const unsigned char *tile[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) tile[t] = a.codes + (size_t)(min(rg * RT + t, a.n_rt - 1) * a.nbp) * (CH * 1024);
  const unsigned char *xbytes = reinterpret_cast<const unsigned char *>(a.x) - 8192;
  const u32 l16[2] = {(u32)lane * 16u, (u32)lane * 16u};
  auto fetch = [&](int b, int slot) __attribute__((always_inline)) {
    const u32 base = ldsb + (u32)(ring + slot * stage);
    const u32 coff = (u32)(b >> 1) * (CH * 1024) + (u32)((b & 1) * (BITS == 3 ? 1024 : 2048));
#pragma unroll
    for (int t = 0; t < RT; ++t)        // 3-bit: chunks 0, 1 or 1, 2 (the middle one holds a half of either block)
      loads_to_lds<2>(tile[t] + coff, l16, base + (u32)(np * 256 + t * 2048));
    const unsigned char *src = xbytes + (size_t)b * 256;
    const int left = a.d_in - b * 128;
    u32 off[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) off[i] = xoff[i];
    if (left < 128) {                   // columns past the end of the row: unit 0 instead, cleared below
#pragma unroll
      for (int i = 0; i < NX; ++i) off[i] = xoct[i] * 8 < left ? xoff[i] : xoff[i] - (u32)xoct[i] * 16u;
    }
#pragma unroll
    for (int i = 0; i < NX; i += 4) loads_to_lds<(NX < 4 ? NX : 4)>(src, off + i, base + (u32)(i * 1024));
  };
  // ---- weak indices; they are back while the first blocks are on their way, and the gathers go out ----
  for (int q = w; q * 256 < a.kp; q += W) {
    const u32 io = (u32)min(q * 256 + lane * 4, a.kp - 4) * 4u;
    load_to_lds(a.weak_idx, io, ldsb + (u32)(a.off_idx + q * 1024));
  }
  for (int d = 0; d < D; ++d)
    if (b0 + d < b1) fetch(b0 + d, d);

  // ---- scales of the workgroup's rows, all groups: two groups per load ----
  for (int q = w; q < RT * ((a.n_groups + 1) >> 1); q += W) {
    const int t = RT == 1 ? 0 : q & 1, gp = RT == 1 ? q : q >> 1;
    const int g = min(2 * gp + kg, a.n_groups - 1), row = min((rg * RT + t) * 32 + n32, a.d_out_pad - 1);
    const u32 off = ((u32)g * (u32)a.d_out_pad + (u32)row) * 4u;
    dword_to_lds(a.sz, off, ldsb + (u32)(a.off_sz + (t * ((a.n_groups + 1) & ~1) + 2 * gp) * 128));
  }
  const int kunits = a.kp >> 3, ksteps = (kunits + 1) >> 1;
  u32x4 wa[RT];                          // the weights of the wave's first k-step of weak columns
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int u = 2 * w + kg;
    wa[t] = (u32x4){0u, 0u, 0u, 0u};
    if (kunits > 0) wa[t] = a.weak_w[(size_t)min((rg * RT + t) * 32 + n32, a.d_out_pad - 1) * kunits + (u < kunits ? u : 0)];
  }
  wait_loads<0>();                       // the first blocks too: the wave could do nothing without them
  __syncthreads();
  // ---- the gathers x[n][idx[t]] go out, as the dwords that hold them; they wait in LDS for the end ----
  const int *idx = reinterpret_cast<const int *>(lds + a.off_idx);
  const int pairs = a.kp << a.lg_tok;    // element e: token e & (np - 1), weak column e >> lg_tok
  for (int e0 = w * 64; e0 < pairs; e0 += 64 * W) {
    const int e = min(e0 + lane, pairs - 1), n = e & (np - 1);
    const int j = idx[e >> a.lg_tok];
    const u32 at = ((u32)(n < a.ntok ? n : 0) * (u32)a.d_in + (u32)(j >= 0 ? j : 0)) * 2u;
    dword_to_lds(a.x, at & ~3u, ldsb + (u32)(a.off_xd + e0 * 4));
  }

  Magic M;
  M.init();
  f16_t tot[RT], acc[RT], zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
  for (int t = 0; t < RT; ++t) tot[t] = zero;
  const int nm = n32 & (np - 1);
  const u32 xsw = (u32)nm * 256u + (u32)((kg ^ (nm & 15)) << 4);
  int slot = 0, g = b0 / a.bpg, gpos = b0 - g * a.bpg;
  // The weak columns of a block are the next ones of the ascending list: a quarter wave clears one of them for 16 tokens,
  // four at a time.  (rank: the first of them; next: the quarter's one, read a block ahead.)
  int rank = 0;
  for (int t0 = 0; t0 < a.k; t0 += 64) rank += __builtin_popcountll(__ballot(t0 + lane < a.k && idx[min(t0 + lane, a.k - 1)] < b0 * 128));
  auto next_weak = [&]() __attribute__((always_inline)) {
    const int t = rank + (lane >> 4);
    return t < a.k ? idx[t] : 0x7fffffff;
  };
  int next = next_weak();
  float zrow[RT];
  auto szof = [&](int t, int gg) __attribute__((always_inline)) {
    return reinterpret_cast<const u32 *>(lds + a.off_sz) + (t * ((a.n_groups + 1) & ~1) + gg) * 32;
  };
#pragma unroll
  for (int t = 0; t < RT; ++t) zrow[t] = half_hi(szof(t, min(g, a.n_groups - 1))[n32]);
  for (int b = b0; b < b1; ++b) {
    if (b + 1 < b1) wait_loads<kPer>();           // the next block's may be in flight
    else wait_loads<0>();
    unsigned char *st = lds + ring + slot * stage;
    // the codes are asked for before the weak columns are cleared
    u32x4 cv[RT][2];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const unsigned char *cs = st + np * 256 + t * 2048 + lane * 16;
      cv[t][0] = *reinterpret_cast<const u32x4 *>(cs);
      cv[t][1] = *reinterpret_cast<const u32x4 *>(cs + 1024);
    }
    auto clear = [&](int col) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < (np + 15) / 16; ++i) {
        const int n = ((lane & 15) + 16 * i) & (np - 1);
        reinterpret_cast<unsigned short *>(st)[n * 128 + ((((col >> 3) ^ (n & 15)) << 3) + (col & 7))] = 0;
      }
    };
    for (;;) {
      const bool mine = next < (b + 1) * 128;
      if (mine) clear(next - b * 128);
      const int cleared = __builtin_popcountll(__ballot(mine)) >> 4;
      rank += cleared;
      next = next_weak();
      if (cleared < 4) break;
    }
    const int left = a.d_in - b * 128;
    if (left < 128)                               // columns past the end of the row
      for (int c = left + (lane >> 4); c < 128; c += 4) clear(c);
    u32 wd[RT][8], nb[RT][8], nr[RT];
    bool rest = false;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const u32x4 v0 = cv[t][0], v1 = cv[t][1];
      if (BITS == 4) {
        wd[t][0] = v0.x; wd[t][1] = v0.y; wd[t][2] = v0.z; wd[t][3] = v0.w;
        wd[t][4] = v1.x; wd[t][5] = v1.y; wd[t][6] = v1.z; wd[t][7] = v1.w;
      } else {
        const bool h = b & 1;
        wd[t][0] = h ? v0.z : v0.x; wd[t][1] = h ? v0.w : v0.y; wd[t][2] = h ? v1.x : v0.z;
        wd[t][3] = h ? v1.y : v0.w; wd[t][4] = h ? v1.z : v1.x; wd[t][5] = h ? v1.w : v1.y;
        wd[t][6] = wd[t][7] = 0u;
      }
      const float z = zrow[t], z1 = __builtin_amdgcn_fmed3f(__builtin_rintf(z), -1024.f, 1024.f);
      const u32 zz = pk_dup(-z1);
#pragma unroll
      for (int o = 0; o < 8; ++o) nb[t][o] = pk_sub(zz, M.m[o]);
      nr[t] = pk_dup(z1 - z);
      rest |= z != z1;
    }
    const bool wrap = gpos + 1 == a.bpg;
    const int gn = wrap && g + 1 < a.n_groups ? g + 1 : g;
    gpos = wrap ? 0 : gpos + 1;
#pragma unroll
    for (int t = 0; t < RT; ++t) zrow[t] = half_hi(szof(t, gn)[n32]);       // of the next block
    FewSteps<BITS, RT, 0>::run(wd, st, xsw, M, nb, acc, zero);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const u32 *szg = szof(t, g);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32x4 s4 = *reinterpret_cast<const u32x4 *>(szg + 8 * q + 4 * kg);
        const float sc[4] = {half_lo(s4.x), half_lo(s4.y), half_lo(s4.z), half_lo(s4.w)};
#pragma unroll
        for (int e = 0; e < 4; ++e) tot[t][4 * q + e] = __builtin_fmaf(sc[e], acc[t][4 * q + e], tot[t][4 * q + e]);
      }
    }
    if (__ballot(rest) != 0ull) {        // what the rounded zero points lack: (rint z - z) times the sum of the block's x
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const h8_t r8 = __builtin_bit_cast(h8_t, (u32x4){nr[t], nr[t], nr[t], nr[t]});
        f16_t e16 = zero;
#pragma unroll
        for (int S = 0; S < 8; ++S) e16 = mma(r8, *reinterpret_cast<const h8_t *>(st + (xsw ^ (S << 5))), e16);
        const u32 *szg = szof(t, g);
#pragma unroll
        for (int r = 0; r < 16; ++r) tot[t][r] = __builtin_fmaf(half_lo(szg[8 * (r >> 2) + 4 * kg + (r & 3)]), e16[r], tot[t][r]);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slot has been read
    if (b + D < b1) fetch(b + D, slot);
    slot = slot + 1 == D ? 0 : slot + 1;
    g = gn;
  }
  // ---- weak columns: the gathered values out of their dwords, then a few k-steps ----
  unsigned short *xw = reinterpret_cast<unsigned short *>(lds + a.off_xw);
  wait_loads<0>();
  for (int e0 = w * 64; e0 < pairs; e0 += 64 * W) {
    const int e = e0 + lane;
    if (e < pairs) {
      const int n = e & (np - 1), j = idx[e >> a.lg_tok];
      const u32 d = reinterpret_cast<const u32 *>(lds + a.off_xd)[e], at = (u32)(n < a.ntok ? n : 0) * (u32)a.d_in + (u32)(j >= 0 ? j : 0);
      xw[n * a.kp + (e >> a.lg_tok)] = j >= 0 ? (unsigned short)(d >> (16 * (at & 1u))) : (unsigned short)0;
    }
  }
  __syncthreads();
  for (int s = w; s < ksteps; s += W) {
    const int u = 2 * s + kg;
    const bool in = u < kunits;
    const u32x4 z4 = {0u, 0u, 0u, 0u};
    const u32x4 bv = *reinterpret_cast<const u32x4 *>(xw + nm * a.kp + (in ? u : 0) * 8);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const u32x4 av = s == w ? wa[t] : a.weak_w[(size_t)min((rg * RT + t) * 32 + n32, a.d_out_pad - 1) * kunits + (in ? u : 0)];
      tot[t] = mma(__builtin_bit_cast(h8_t, in ? av : z4), __builtin_bit_cast(h8_t, in ? bv : z4), tot[t]);
    }
  }
  // ---- the waves' results, added in a fixed order ----
  float *red = reinterpret_cast<float *>(lds);
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[((w * RT + t) * 16 + r) * 65 + lane] = tot[t][r];      // odd pitch: the sums read down a column
  __syncthreads();
  for (int e = tid; e < a.ntok * 32 * RT; e += (int)blockDim.x) {
    const int row = e & 31, t = RT == 1 ? 0 : (e >> 5) & 1, nn = e >> (RT == 1 ? 5 : 6);
    const int r = 4 * (row >> 3) + (row & 3), ln = nn + 32 * ((row >> 2) & 1);
    float v = 0.f;
    for (int q = 0; q < W; ++q) v += red[((q * RT + t) * 16 + r) * 65 + ln];
    const int grow = (rg * RT + t) * 32 + row;
    if (grow < a.d_out) a.y[(size_t)nn * a.d_out + grow] = (_Float16)v;
  }
}

typedef void (*few_fn)(const FewArgs);
template <int BITS, int RT>
few_fn pick_few_nx(int nx) {
  if (nx == 1) return owq_tile_few<BITS, RT, 1>;
  if (nx == 2) return owq_tile_few<BITS, RT, 2>;
  return nx == 4 ? owq_tile_few<BITS, RT, 4> : owq_tile_few<BITS, RT, 8>;
}
few_fn pick_few(int bits, int rt, int nx) {
  if (bits == 3) return rt == 2 ? pick_few_nx<3, 2>(nx) : pick_few_nx<3, 1>(nx);
  return rt == 2 ? pick_few_nx<4, 2>(nx) : pick_few_nx<4, 1>(nx);
}

}  // namespace

int prepare_tile_few_kernels(const owq_layer_info_t &g, int32_t lds_limit) {
  for (int rt = 1; rt <= 2; ++rt)
    for (int nx = 1; nx <= 8; nx *= 2) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_few(g.bits, rt, nx)),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kFewLds < lds_limit ? kFewLds : lds_limit);
      if (e != hipSuccess) return (int)e;
    }
  return (int)hipSuccess;
}

int launch_tile_few(const owq_layer_info_t &g, void *blob, int32_t lds_limit, const void *x, void *y, int32_t ntok, void *stream) {
  if (ntok < 1 || ntok > 32 || (reinterpret_cast<uintptr_t>(x) & 15) != 0 || (g.d_in & 7) != 0 || g.kp > kFewKp) return -1;
  int lg_tok = 2;
  while ((1 << lg_tok) < ntok) ++lg_tok;
  const int np = 1 << lg_tok, waves = np > 16 ? 4 : 8, nblk = (g.d_in + kBlockCols - 1) / kBlockCols;
  auto up = [](int n) { return (n + 1023) & ~1023; };      // what loads of 1 KB fill
  const int xw = up(np * g.kp * 2), xd = up(np * g.kp * 4), idx = up(g.kp * 4);
  // One or two row tiles per workgroup, and whether this kernel at all: a wave's blocks run one after the other (us per
  // block below), so layers with few rows and many columns, and layers of several rounds of workgroups, are better off
  // with their columns spread over workgroups.  Measured in us, this kernel / the others: 5120 x 5120, 16 tokens 9.0 / 14.1;
  // 13824 x 5120 15.1 / 21.0; 5120 x 13824 19.8 / 22.3; 4096 x 4096, 5 tokens 7.0 / 9.7; 16384 x 4096 rows, 32 tokens
  // 17.4 / 22.2; 4096 rows x 16384 columns, 24 tokens 36.2 / 23.2.
  const float mb = (float)g.n_rt * g.nbp * 64 * g.chunks * 16 / 1e6f;
  float best = 15.f + mb / 4.2f;
  // (several workgroups per row tile: whole blocks and groups of 128 2^n only.  Layers with others went by that cost too and took three
  // launches: 7000 -> 2048 at 4 / 16 tokens 15.2 / 15.6 us, 10.3 / 11.9 so; 9000 -> 3000 16.3 / 16.5, 12.3 / 14.1; 7680 -> 2048 in
  // groups of 384 15.7 / 16.2, 11.1 / 12.7.  8192 -> 4096, 3-bit, 12.7 / 16.0,
  // 11.4 / 12.6; 4096 -> 512 at 8 7.6, 6.7; 6144 -> 1024 stays at 8.1 at 4 tokens, 8.7 here, and takes 9.8 instead of 11.3 at 16; one token of 8192 -> 4096 10.6, 11.1)
  const float spread = (ntok > 8 ? 10.5f : ntok > 2 ? 10.f : 8.5f) + 0.38f * mb;
  const bool spreads = g.d_in % kBlockCols == 0 && (g.n_groups <= 1 || (g.group_size & (g.group_size - 1)) == 0);
  if (ntok <= 16 && spreads && best > spread) best = spread;
  int rt = 0, ring = 0, sz = 0, total = 0;
  for (int r = 1; r <= 2; ++r) {
    const int wgs = (g.n_rt + r - 1) / r, rg_bytes = waves * kFewDepth * (np * 256 + r * 2048);
    const int red = waves * r * 16 * 65 * 4;                // the sums reuse the ring
    const int ri = up(rg_bytes > red ? rg_bytes : red), si = up(r * ((g.n_groups + 1) & ~1) * 128);
    if (ri + si + xw + xd + idx > (kFewLds < lds_limit ? kFewLds : lds_limit)) continue;
    const float block = waves == 8 ? (r == 1 ? 1.0f : 1.8f) : (r == 1 ? 0.95f : 1.5f);
    const float us = 5.5f + ((wgs + 255) / 256) * ((nblk + waves - 1) / waves) * block;
    if (us < best) { best = us; rt = r; ring = ri; sz = si; total = ri + si + xw + xd + idx; }
  }
  if (rt == 0) return -1;
  uint8_t *base = static_cast<uint8_t *>(blob);
  FewArgs a;
  a.codes = base + g.off_codes;
  a.sz = reinterpret_cast<const u32 *>(base + g.off_sz);
  a.weak_idx = reinterpret_cast<const int *>(base + g.off_weak_idx);
  a.weak_w = reinterpret_cast<const u32x4 *>(base + g.off_weak_w);
  a.x = static_cast<const _Float16 *>(x);
  a.y = static_cast<_Float16 *>(y);
  a.d_in = g.d_in; a.d_out = g.d_out; a.d_out_pad = g.d_out_pad; a.n_rt = g.n_rt; a.ntok = ntok; a.nbp = g.nbp;
  a.nblk = nblk;
  a.n_groups = g.n_groups;
  a.bpg = g.group_size ? g.group_size / kBlockCols : g.nblk;
  a.k = g.k; a.kp = g.kp; a.lg_tok = lg_tok;
  a.off_sz = ring;
  a.off_xw = ring + sz;
  a.off_xd = a.off_xw + xw;
  a.off_idx = a.off_xd + xd;
  hipLaunchKernelGGL(pick_few(g.bits, rt, np / 4), dim3((unsigned)((g.n_rt + rt - 1) / rt)), dim3((unsigned)(waves * 64)),
                     (size_t)total, static_cast<hipStream_t>(stream), a);
  return (int)hipGetLastError();
}

}  // namespace owq
