// Line screen of the one-sided sweeps, and the screened forward sweep.
//
// A one-sided quantity sums (or differentiates) one penalty side over every
// outage x line element: the lower penalties max(|C| - R - fmax, 0) for f_hi,
// the upper ones max(|C| + R - fmax, 0) for f_lo (Sec. III-A eqs. (slack-Sc),
// (slack-sagg); Sec. III-C eq. (IBP)).  Post-outage flows are
// C = c_l + Lam c_c and R = r_l + |Lam| r_c (Sec. II-C, eq. ctg flow
// simplified), so with w_k = |c_c| - r_c (lower) or |c_c| + r_c (upper) for
// the outaged line of outage k, every element of line l obeys
//   |C| - R - fmax <= (|c_l| - (r_l + fmax)) + |Lam_lk| max(w_k, 0),
//   |C| + R - fmax <= (|c_l| + (r_l - fmax)) + |Lam_lk| w_k.
// A line on which the right-hand side stays below zero for every outage and
// every box of a tile holds no active element there, and contributes nothing.
// In sub-boxes few lines can (2000 buses, 4096 sub-boxes: 19% of the
// (4-box tile, line) pairs for the lower penalties; at the boxes' centre
// points 39% for the upper ones).
//
// K5w takes per tile and outage the largest max(w_k, 0) over the tile's
// boxes; K5s, per tile and line, the largest |Lam_lk| W_k over the outages
// (one multiply and one max per factor and tile, 16 or 4 tiles per block
// sharing each factor load) and marks the line where base + that > -margin.
// margin is 32 float32 unit roundoffs of the largest magnitude either test adds
// (the screen's own bound and the sweep's test take 12 between them), so no
// line with an active element goes unmarked.  The radii and limits are those
// of the sweep the screen serves: the backward's unpadded ones, or the
// forward's padded r' and fmax -/+ r' (which only make its penalties
// smaller on the lower side; on the upper side they enter the bound).  Marked
// lines get their tile record (the four boxes' centres and radius terms),
// which the sweeps read by scalar loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>

#include "ibp_device.h"
#include "ibp_devfun.h"
#include "ibp_kernels.h"
#include "ibp_lanes.h"

namespace ibp {

constexpr int kScreenChunk = 64;  // outages per LDS chunk of the screen

// Tiles per screen block: sixteen share every factor load where outages are many (1024
// boxes at 2000 buses, with the split below 0.17 ms; four and no split 0.42) or
// blocks too; with few outages the marks are the work, and four finish earlier (14160
// boxes at 20 buses 13 against 33 us).
//
// Outage ranges a line block and tile group is split over when those alone leave the
// chip half idle (seven blocks fit a CU); k5s_mark then joins the ranges' masks.  4096 boxes at
// 2000 buses 0.79 -> 0.50 ms and 0.07 for the join, 2533 at 529 buses 78 -> 33 us and 10, 8
// at 2000 buses 600 -> 30 us.
constexpr int kScreenBlocks = 1792;
inline int screen_tiles(const DevNet& net, const WsLayout& lay) {
  const int64_t wide = ((int64_t)lay.k5s_tiles + 15) / 16 * ((net.Lp + 255) / 256);
  return wide >= 512 || (wide >= 64 && net.K >= 1024) ? 16 : 4;
}
inline int screen_splits(const DevNet& net, const WsLayout& lay) {
  const int g = screen_tiles(net, lay);
  const int64_t blocks = (int64_t)((lay.k5s_tiles + g - 1) / g) * ((net.Lp + 255) / 256);
  if (2 * blocks > kScreenBlocks) return 1;
  return (int)std::max<int64_t>(1, std::min<int64_t>(kScreenBlocks / blocks, lay.cm_groups));
}

// The per-outage (centre, radius) the sweep of `mode` uses: the backward's
// (centre, unpadded radius) pairs, or the forward's (centre, padded r').
template <int MODE>
__device__ __forceinline__ float2 outage_cr(const DevNet& net, void* ws, const WsLayout& lay, int64_t b, int k) {
  if (MODE == kScreenBackwardLower) return ws_ptr<float2>(ws, lay.cb)[b * net.K + k];
  const int4 d = ws_ptr<int4>(ws, lay.ctg)[b * net.K + k];
  return make_float2(__int_as_float(d.y), __int_as_float(d.z));
}

// The per-line radius term of the sweep's test for box b: r + fmax
// (backward), or the forward sweep's padded g = r' + fmax and
// h = r' - fmax, each raised by the line's construction error times the box's
// largest outage magnitude exactly as that sweep forms them.
template <int MODE>
__device__ __forceinline__ float line_term(const DevNet& net, void* ws, const WsLayout& lay, int64_t b, int l,
                                           float fc) {
  if (MODE == kScreenBackwardLower) return (float)ws_ptr<double>(ws, lay.lrf)[b * net.L + l] + fc;
  const double* bs = ws_ptr<double>(ws, lay.box) + b * kBoxSlots;
  const float vmax = __uint_as_float(*reinterpret_cast<const unsigned int*>(bs + kVmax));
  const float ex = next_up_f32(net.line_eps[l] * vmax);
  const float v = ws_ptr<float>(ws, MODE == kScreenForwardLower ? lay.lg : lay.lh)[b * net.Lp + l];
  return add_ru(v, ex);
}

// The forward sweep's padded g of box b and line l (the lower penalties' term
// of a two-sided sweep), formed as K3b forms it.
__device__ __forceinline__ float line_g(const DevNet& net, void* ws, const WsLayout& lay, int64_t b, int l) {
  const double* bs = ws_ptr<double>(ws, lay.box) + b * kBoxSlots;
  const float vmax = __uint_as_float(*reinterpret_cast<const unsigned int*>(bs + kVmax));
  return add_ru(ws_ptr<float>(ws, lay.lg)[b * net.Lp + l], next_up_f32(net.line_eps[l] * vmax));
}

// K5w: per tile (grid x: a call may have more than the 65535 of the other two) and
// outage W (zero past the last outage); per tile and block of 256 outages the largest
// |c_c| + r_c, for the margin.
template <int MODE>
__global__ __launch_bounds__(256) void k5w_tile_max(DevNet net, void* ws, WsLayout lay, int64_t n_box) {
  constexpr int S = kScreenBoxes;
  __shared__ unsigned zs[4];
  const int k = blockIdx.y * 256 + threadIdx.x;
  const int64_t t = blockIdx.x;
  float wv = 0.0f, z = 0.0f;
  if (k < net.K) {
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int64_t b = t * S + i;
      if (b < n_box) {
        const float2 v = outage_cr<MODE>(net, ws, lay, b, k);
        wv = fmaxf(wv, MODE >= kScreenForwardUpper ? fabsf(v.x) + v.y : fabsf(v.x) - v.y);
        z = fmaxf(z, fabsf(v.x) + v.y);
      }
    }
  }
  if (k < net.Kp) ws_ptr<float>(ws, lay.sw)[t * net.Kp + k] = wv;
  // non-negative floats order like their bit patterns
  const unsigned zb = wave_max_u32(__float_as_uint(z));
  if ((threadIdx.x & 63) == 0) zs[threadIdx.x >> 6] = zb;
  __syncthreads();
  if (threadIdx.x == 0)
    ws_ptr<float>(ws, lay.sz)[t * lay.k5w_bx + blockIdx.y] =
        __uint_as_float(max(max(zs[0], zs[1]), max(zs[2], zs[3])));
}

// What |Lam| W has to exceed for an element of the line in one of the tile's boxes to
// be active (lowered by the margin of the float32 roundings): z is the tile's largest
// |c_c| + r_c.
template <int MODE>
__device__ __forceinline__ float line_threshold(const DevNet& net, void* ws, const WsLayout& lay, int64_t n_box,
                                                int64_t t, int l, bool lon, float z, float fc, float amax) {
  constexpr int S = kScreenBoxes;
  const float* lc = ws_ptr<float>(ws, lay.lc);
  float base = -FLT_MAX, sc = 0.0f;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const int64_t b = t * S + i;
    if (lon && b < n_box) {
      const float c = lc[b * net.Lp + l], r = line_term<MODE>(net, ws, lay, b, l, fc);
      base = fmaxf(base, MODE >= kScreenForwardUpper ? fabsf(c) + r : fabsf(c) - r);
      sc = fmaxf(sc, fabsf(c) + fabsf(r));
    }
  }
  const float margin = 0x1p-19f * (sc + amax * z);
  return lon ? -margin - base : INFINITY;
}

// One line's mark in one tile and, if it is marked, its record: every lane of the
// block's waves calls it with its own line.
template <int MODE>
__device__ __forceinline__ void mark_line(const DevNet& net, void* ws, const WsLayout& lay, int64_t n_box, int64_t t,
                                          int l, bool flag, float fc) {
  constexpr int S = kScreenBoxes;
  static_assert(S == 4, "a tile's line record holds four boxes");
  // a box past the end gets a record that never tests active
  constexpr float kOff = MODE >= kScreenForwardUpper ? -INFINITY : INFINITY;
  const float* lc = ws_ptr<float>(ws, lay.lc);
  const int words = net.Lp / 64, word = l >> 6;
  const uint64_t bits = __builtin_amdgcn_ballot_w64(flag);
  if ((threadIdx.x & 63) == 0 && word < words) ws_ptr<uint64_t>(ws, lay.smask)[t * words + word] = bits;
  if (!flag) return;
  float cv[S], rv[S], gv[S];
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const int64_t b = t * S + i;
    cv[i] = 0.0f;
    rv[i] = kOff;
    gv[i] = INFINITY;
    if (b < n_box) {
      cv[i] = lc[b * net.Lp + l];
      rv[i] = line_term<MODE>(net, ws, lay, b, l, fc);
    }
  }
  float4* rec = reinterpret_cast<float4*>(ws_ptr<float>(ws, lay.srec) + ((size_t)t * net.Lp + l) * kScreenRecFloats);
  rec[0] = make_float4(cv[0], cv[1], cv[2], cv[3]);
  rec[1] = make_float4(rv[0], rv[1], rv[2], rv[3]);
  if (MODE == kScreenForwardBoth) {
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (t * S + i < n_box) gv[i] = line_g(net, ws, lay, t * S + i, l);
    rec[2] = make_float4(gv[0], gv[1], gv[2], gv[3]);
  }
  if (MODE == kScreenBackwardLower) {
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (t * S + i < n_box) ws_ptr<uint64_t>(ws, lay.lcnt)[(t * S + i) * net.Lp + l] = 0ull;
  }
}

// K5s: one line per lane, G tiles per block, the tiles' W staged in LDS
// kScreenChunk outages at a time; outage range blockIdx.z of gridDim.z.  A line is
// marked per group of 256 << cm_shift outages, the sweeps' chunks: a line that only
// some outages move over its limit is walked for their chunks alone (8192 centre points
// at 2000 buses: 35% of the lines are marked, 21% of the lines and chunks; their sweep
// 3.4 -> 2.2 ms, that of the boxes 1.6 -> 1.05).  Waits for the factors and for W bound
// the kernel: with seven waves per SIMD (72 registers, thresholds in LDS) 8192 boxes take
// 1.04 ms, with four 1.35.
template <int MODE, int G>
__global__ __launch_bounds__(256, 7) void k5s_screen(DevNet net, void* ws, WsLayout lay, int64_t n_box, int k_per) {
  static_assert(G % 4 == 0, "tiles are read from LDS as float4");
  __shared__ __align__(16) float wsh[kScreenChunk][G];
  __shared__ float tsh[G][256];   // the thresholds (a group's end reads them)
  float* zsh = &wsh[0][0];        // the tiles' margin scales, before the first chunk
  const int tid = threadIdx.x, lane = tid & 63;
  const int l = blockIdx.x * 256 + tid;
  const bool lon = l < net.L;
  const int words = net.Lp / 64, word = l >> 6;
  const int64_t tile0 = (int64_t)blockIdx.y * G;
  const int ntile = (int)min<int64_t>(G, lay.k5s_tiles - tile0);
  const int kbeg = blockIdx.z * k_per, kend = min(net.K, kbeg + k_per);
  const float* W = ws_ptr<float>(ws, lay.sw) + tile0 * net.Kp;
  if (tid < G) {
    float z = 0.0f;
    if (tid < ntile)
      for (int j = 0; j < lay.k5w_bx; ++j) z = fmaxf(z, ws_ptr<float>(ws, lay.sz)[(tile0 + tid) * lay.k5w_bx + j]);
    zsh[tid] = z;
  }
  __syncthreads();
  const float fc = lon ? net.fmax_c32[l] : 0.0f, amax = lon ? net.lam_max[l] : 0.0f;
  float m[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = 0.0f;
    tsh[g][tid] = g < ntile ? line_threshold<MODE>(net, ws, lay, n_box, tile0 + g, l, lon, zsh[g], fc, amax) : INFINITY;
  }
  unsigned any = 0u;  // bit g: marked in some group
  const int group = 256 << lay.cm_shift;
  const float* lam = net.lodf + min(l, net.Lp - 1);
  for (int k0 = kbeg; k0 < kend; k0 += kScreenChunk) {
    const int nk = min(kScreenChunk, kend - k0);
    __syncthreads();
    for (int idx = tid; idx < kScreenChunk * G; idx += 256) {
      const int kk = idx % kScreenChunk, g = idx / kScreenChunk;
      wsh[kk][g] = (g < ntile && kk < nk) ? W[(size_t)g * net.Kp + k0 + kk] : 0.0f;
    }
    __syncthreads();
    // |Lam| W: the outaged line's own factor is NaN, and fmaxf keeps m there;
    // rows past the chunk's end read its last row against W = 0
    for (int kk = 0; kk < nk; kk += 8) {
      float a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = fabsf(lam[(size_t)(k0 + min(kk + u, nk - 1)) * net.Lp]);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
#pragma unroll
        for (int g4 = 0; g4 < G / 4; ++g4) {
          const float4 wv = *reinterpret_cast<const float4*>(&wsh[kk + u][4 * g4]);
          m[4 * g4 + 0] = fmaxf(m[4 * g4 + 0], a[u] * wv.x);
          m[4 * g4 + 1] = fmaxf(m[4 * g4 + 1], a[u] * wv.y);
          m[4 * g4 + 2] = fmaxf(m[4 * g4 + 2], a[u] * wv.z);
          m[4 * g4 + 3] = fmaxf(m[4 * g4 + 3], a[u] * wv.w);
        }
      }
    }
    const int k1 = k0 + kScreenChunk;
    if (k1 < kend && k1 % group != 0) continue;
    uint64_t* cm = ws_ptr<uint64_t>(ws, lay.cmask) + ((size_t)tile0 * lay.cm_groups + k0 / group) * words + word;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const bool on = m[g] > tsh[g][tid];
      const uint64_t bits = __builtin_amdgcn_ballot_w64(on);
      if (lane == 0 && g < ntile && word < words) cm[(size_t)g * lay.cm_groups * words] = bits;
      any |= on ? 1u << g : 0u;
      m[g] = 0.0f;
    }
  }
  if (gridDim.z > 1) return;
  for (int g = 0; g < ntile; ++g) mark_line<MODE>(net, ws, lay, n_box, tile0 + g, l, (any >> g) & 1u, fc);
}

// The marks of a screen that was split over the outages: one tile per block row.
template <int MODE>
__global__ __launch_bounds__(256) void k5s_mark(DevNet net, void* ws, WsLayout lay, int64_t n_box) {
  const int l = blockIdx.x * 256 + threadIdx.x;
  const int64_t t = blockIdx.y;
  const int words = net.Lp / 64, word = min(l >> 6, words - 1);
  const uint64_t* cm = ws_ptr<uint64_t>(ws, lay.cmask) + (size_t)t * lay.cm_groups * words + word;
  uint64_t any = 0;
#pragma unroll 8
  for (int j = 0; j < lay.cm_groups; ++j) any |= cm[(size_t)j * words];
  mark_line<MODE>(net, ws, lay, n_box, t, l, l < net.L && ((any >> (l & 63)) & 1), l < net.L ? net.fmax_c32[l] : 0.0f);
}

template <int MODE>
static void launch_screen_mode(const DevNet& net, int64_t n_box, void* ws, const WsLayout& lay, hipStream_t s) {
  const int z = screen_splits(net, lay), g = screen_tiles(net, lay);
  const int group = 256 << lay.cm_shift;
  const int k_per = ((net.K + z - 1) / z + group - 1) / group * group;
  const unsigned gx = (net.Lp + 255) / 256, gz = (unsigned)((net.K + k_per - 1) / k_per);
  hipLaunchKernelGGL(k5w_tile_max<MODE>, dim3(lay.k5s_tiles, lay.k5w_bx), dim3(256), 0, s, net, ws, lay, n_box);
  const dim3 grid(gx, (lay.k5s_tiles + g - 1) / g, gz);
  if (g == 16)
    hipLaunchKernelGGL((k5s_screen<MODE, 16>), grid, dim3(256), 0, s, net, ws, lay, n_box, k_per);
  else
    hipLaunchKernelGGL((k5s_screen<MODE, 4>), grid, dim3(256), 0, s, net, ws, lay, n_box, k_per);
  // (a split screen has at most kScreenBlocks / 2 tile groups: far below 65535 rows)
  if (gz > 1) hipLaunchKernelGGL(k5s_mark<MODE>, dim3(gx, lay.k5s_tiles), dim3(256), 0, s, net, ws, lay, n_box);
}

void launch_line_screen(const DevNet& net, int64_t n_box, void* ws, const WsLayout& lay, int mode, hipStream_t s) {
  if (mode == kScreenBackwardLower)
    launch_screen_mode<kScreenBackwardLower>(net, n_box, ws, lay, s);
  else if (mode == kScreenForwardLower)
    launch_screen_mode<kScreenForwardLower>(net, n_box, ws, lay, s);
  else if (mode == kScreenForwardUpper)
    launch_screen_mode<kScreenForwardUpper>(net, n_box, ws, lay, s);
  else
    launch_screen_mode<kScreenForwardBoth>(net, n_box, ws, lay, s);
}

// K3p: the one-sided forward sweep over the marked lines.  A wave holds 64 Q
// outages (lanes) of one tile's boxes and walks the tile's marked lines (the
// same walk as the backward's K5p); each element is k3_elem's, bit for bit
// (the same float32 operations on the same values), and each line's Q
// elements per box are summed in float32 (depth 2, within the depth-3 sums
// the padding of the outage-penalty total allows) and added in float64.
// Per (box, chunk of 64 Q outages, line segment) one float64 partial, in the slot
// the finalize sums; slots past the last one are cleared.  The lines are walked in
// n_seg segments, a wave each, where tiles and chunks give few waves (sweep_segments).
template <int SIDES, int Q>
__global__ __launch_bounds__(256) void k3p_sweep(DevNet net, void* ws, WsLayout lay, int64_t n_box, int n_chunk,
                                                 int n_tg, int n_seg) {
  constexpr int S = kScreenBoxes;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // unit u = (chunk, group of 4 tiles: one per wave), chunk-major, and the
  // blocks of one XCD (block id mod 8) on consecutive units
  const int U = n_chunk * n_seg * n_tg;
  const int per = (U + 7) / 8;
  const int slot = blockIdx.x >> 3;
  const int u = (blockIdx.x & 7) * per + slot;
  if (slot >= per || u >= U) return;  // the whole block
  const int tile = (u % n_tg) * 4 + w;
  const bool on = tile < lay.k5s_tiles;
  const int seg = (u / n_tg) % n_seg, chunk = u / n_tg / n_seg;
  const int kw = chunk * 64 * Q;
  __shared__ uint64_t smk_all[4][kSparseMaxWords];
  uint64_t* smk = smk_all[w];
  const int per_seg = (net.Lp / 64 + n_seg - 1) / n_seg, word0 = seg * per_seg;
  const int words = min(per_seg, net.Lp / 64 - word0);  // of this segment (may be none)
  if (on) {
    const int group = (kw >> 8) >> lay.cm_shift;  // of this wave's outages
    const uint64_t* mask =
        ws_ptr<uint64_t>(ws, lay.cmask) + ((size_t)tile * lay.cm_groups + group) * (net.Lp / 64) + word0;
    for (int j = lane; j < words; j += 64) smk[j] = mask[j];
  }
  __syncthreads();
  if (!on) return;
  const int64_t b0 = (int64_t)tile * S;
  int64_t bb[S];
#pragma unroll
  for (int i = 0; i < S; ++i) bb[i] = min(b0 + i, n_box - 1);
  // per-lane outage data; lanes past the last outage get r' = inf (their
  // factors are the zero padding, and 0 x inf = NaN fails every test)
  float cc[Q][S], rk[Q][S];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int k = kw + 64 * q + lane;
    const int kq = min(k, net.K - 1);
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int4 d = ws_ptr<int4>(ws, lay.ctg)[bb[i] * net.K + kq];
      cc[q][i] = __int_as_float(d.y);
      rk[q][i] = k < net.K ? __int_as_float(d.z) : INFINITY;
    }
  }
  double acc[S], acc2[S];  // SIDES 3: acc the upper penalties, acc2 the lower
#pragma unroll
  for (int i = 0; i < S; ++i) acc[i] = acc2[i] = 0.0;
  typedef __attribute__((address_space(4))) const float const_float;
  const_float* rec = (const_float*)(ws_ptr<float>(ws, lay.srec) + (size_t)tile * net.Lp * kScreenRecFloats);
  static_assert(64 * Q <= 256, "a chunk must fit the 256-outage row padding");
  const float* __restrict__ lamT = net.lodfT + kw + lane;
  // records: SIDES 1 (centres, g), SIDES 2 (centres, h), SIDES 3 (centres,
  // h, g)
  auto line_step = [&](const float4& c4, const float4& r4, const float4& g4, const float (&x)[Q]) {
    // each record value is read by Q elements' instructions: vector copies
    const float cl[S] = {vcopy(c4.x), vcopy(c4.y), vcopy(c4.z), vcopy(c4.w)};
    const float rl[S] = {vcopy(r4.x), vcopy(r4.y), vcopy(r4.z), vcopy(r4.w)};
    const float gl[S] = {SIDES == 3 ? vcopy(g4.x) : 0.0f, SIDES == 3 ? vcopy(g4.y) : 0.0f,
                         SIDES == 3 ? vcopy(g4.z) : 0.0f, SIDES == 3 ? vcopy(g4.w) : 0.0f};
#pragma unroll
    for (int i = 0; i < S; ++i) {
      float p[Q], p2[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        float a, b;
        k3_elem<SIDES>(x[q], cc[q][i], rk[q][i], cl[i], rl[i], SIDES == 3 ? gl[i] : rl[i], a, b);
        p[q] = SIDES == 1 ? b : a;
        p2[q] = b;
      }
      static_assert(Q == 4, "the float32 sum is written for four outages");
      acc[i] += (double)((p[0] + p[1]) + (p[2] + p[3]));
      if (SIDES == 3) acc2[i] += (double)((p2[0] + p2[1]) + (p2[2] + p2[3]));
    }
  };
  // marked-line walk (wave-uniform): lane i holds mask word wb + i, read out
  // by readlane; each line's loads issued before the previous line's sums
  int j = 0, wb = 0;
  uint64_t bits = 0;
  uint64_t mw = lane < words ? smk[lane] : 0ull;
  auto next = [&]() -> int {
    while (bits == 0) {
      if (j >= words) return -1;
      if (j - wb >= 64) {
        wb += 64;
        mw = wb + lane < words ? smk[wb + lane] : 0ull;
      }
      const int i = j - wb;
      bits = ((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)(mw >> 32), i) << 32) |
             (unsigned)__builtin_amdgcn_readlane((int)(unsigned)mw, i);
      ++j;
    }
    const int l = (word0 + j - 1) * 64 + __builtin_ctzll(bits);
    bits &= bits - 1;
    return l;
  };
  bool pending = false;
  float4 pc4 = make_float4(0.f, 0.f, 0.f, 0.f), pr4 = pc4, pg4 = pc4;
  float px[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) px[q] = 0.0f;
  for (int l = next(); l >= 0; l = next()) {
    const_float* rp = rec + kScreenRecFloats * (size_t)l;
    const float4 c4 = make_float4(rp[0], rp[1], rp[2], rp[3]), r4 = make_float4(rp[4], rp[5], rp[6], rp[7]);
    const float4 g4 = SIDES == 3 ? make_float4(rp[8], rp[9], rp[10], rp[11]) : r4;
    float x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) x[q] = lamT[(size_t)l * net.Kp + 64 * q];
    if (pending) line_step(pc4, pr4, pg4, px);
    pending = true;
    pc4 = c4;
    pr4 = r4;
    pg4 = g4;
#pragma unroll
    for (int q = 0; q < Q; ++q) px[q] = x[q];
  }
  if (pending) line_step(pc4, pr4, pg4, px);
  double2* p3 = ws_ptr<double2>(ws, lay.p3);
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const double t = wave_sum(acc[i]);
    const double t2 = SIDES == 3 ? wave_sum(acc2[i]) : 0.0;
    if (lane == 0 && b0 + i < n_box) {
      p3[(b0 + i) * lay.n_p3 + chunk * n_seg + seg] = SIDES == 1 ? make_double2(0.0, t) : make_double2(t, t2);
      if (chunk == 0 && seg == 0)
        for (int c = n_chunk * n_seg; c < lay.n_p3; ++c) p3[(b0 + i) * lay.n_p3 + c] = make_double2(0.0, 0.0);
    }
  }
}

void launch_screened_forward_sweep(const DevNet& net, int64_t n_box, void* ws, const WsLayout& lay, int sides,
                                   hipStream_t s) {
  const int n_chunk = (net.K + 64 * kSparseQ - 1) / (64 * kSparseQ), n_tg = (lay.k5s_tiles + 3) / 4;
  const int n_seg = sweep_segments(net, n_chunk * n_tg, lay.n_p3 / n_chunk);
  const int per = (n_chunk * n_seg * n_tg + 7) / 8;
  if (sides == 1)
    hipLaunchKernelGGL((k3p_sweep<1, kSparseQ>), dim3(8 * per), dim3(256), 0, s, net, ws, lay, n_box, n_chunk, n_tg,
                       n_seg);
  else if (sides == 2)
    hipLaunchKernelGGL((k3p_sweep<2, kSparseQ>), dim3(8 * per), dim3(256), 0, s, net, ws, lay, n_box, n_chunk, n_tg,
                       n_seg);
  else
    hipLaunchKernelGGL((k3p_sweep<3, kSparseQ>), dim3(8 * per), dim3(256), 0, s, net, ws, lay, n_box, n_chunk, n_tg,
                       n_seg);
}

}  // namespace ibp
