// The outage sweep of many boxes as integer matrix products plus exceptions.
//
// An element's penalty max(|C| + A, 0) (upper) or max(|C| - B, 0) (lower), with
// C = c_l + Lam c_c, A = h_l + |Lam| r_k, B = g_l + |Lam| r_k (Sec. II-C, eq. ctg
// flow simplified; Sec. III-A, eq. slack-Sc), is linear in (Lam, |Lam|) wherever
// the outage changes neither the sign of the line's base flow nor whether the
// penalty is active.  Post-outage flows differ little from base flows on most
// lines, so this holds for all but a few elements (2000 buses, sub-boxes: 0.5%
// of them fail it for either side; 8316 buses: 0.1%).  With a_l in {0, 1} (the
// base flow's own penalty is active) and v_l = a_l sign(c_l), the sum over all
// outages k != the line's own is therefore
//   sum_l a_l (K_l (|c_l| + h_l)) + sum_k c_k (Lam^T v)_k + sum_k r_k (|Lam|^T a)_k
// plus, for the elements where the assumption may fail, the true penalty minus
// the linear one.  (Lower side: -g_l, -r_k and its own a.)
//
// The two contractions run on the integer matrix cores, exactly: Lam is held as
// a multiple of 2^-38 in five balanced base-256 digits, a and v are 0 or +-1, so
// every digit product sum fits in int32.  No floating-point rounding enters
// them; the weighted sums over k are float64.  K L B element evaluations (9.25
// float32 VALU ops each in the dense sweep) become 20 int8 products of the same
// size (two sides, signed and absolute, five digits) at 32 times the VALU's rate.
//
//   KN1  kn_outages  per group of 64 boxes: (c_k, r_k) outage-major, and the
//                    group's largest |c_k| + r_k
//   KN2  kn_lines    per 64 boxes x 32 lines: a, v, the lines' own sums; a scan of
//                    the lines' factors finds the elements that may be exceptional
//                    in a box of the group, which are evaluated in float64
//   KN2p kn_pairs    the (line, box) pairs near a kink, swept densely
//   KN2h kn_heavy    the lines with the largest flows, swept densely
//   KN3  kn_gemm     the digit products and their float64 weighted sums
//
// Error model.  The model's elements use the stored factor rounded to 2^-38
// (exact from 2^-15 on): t moves by at most 2^-39 (|c_k| + r_k), below the
// 2 u32 fmax_l that r'_l carries for float32 roundings this path does not make, as
// long as |c_k| + r_k <= 2^15 fmax; the finalize adds the difference of larger
// flows explicitly (kWmax).  Float64 rounding is bounded by the sums of absolute
// terms written beside the partials (lay.pe).  Both are charged against the
// +-4 u32 by which the finalize scales the totals for float32 sums.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "ibp_device.h"
#include "ibp_devfun.h"
#include "ibp_kernels.h"
#include "ibp_lanes.h"

namespace ibp {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

static_assert(kLinGroup == 64, "a lane per box");

// The factor as the digit products hold it: a multiple of 2^-38, a float32 value.
__device__ __forceinline__ float lin_factor(float lam) { return rintf(lam * 0x1p38f) * 0x1p-38f; }

// max(x, 0) and max(-x, 0) in one instruction (fmax would first canonicalise an
// operand whose sign bit was flipped as an integer); NaN gives 0.
__device__ __forceinline__ double relu(double x) {
  double r;
  __asm__("v_max_f64 %0, %1, 0" : "=v"(r) : "v"(x));
  return r;
}
__device__ __forceinline__ double relu_neg(double x) {
  double r;
  __asm__("v_max_f64 %0, -%1, 0" : "=v"(r) : "v"(x));
  return r;
}

__device__ __forceinline__ double flip_sign(double x, unsigned sign) {
  const unsigned long long v = (unsigned long long)__double_as_longlong(x);
  return __longlong_as_double((long long)(v ^ ((unsigned long long)sign << 32)));
}

// Outage that lane i of a 64-lane sample stands for.
__device__ __forceinline__ int lin_sample(int K, int i) { return K >= 64 ? (int)((int64_t)i * K / 64) : min(i, K - 1); }

// Digit planes of the outage factors in the operand order of
// v_mfma_i32_32x32x32_i8: [32 outages][32 lines][5 digits][64 lanes][16 bytes],
// lane i holding row i % 32, columns 16 (i / 32) ..+15.  `dig`: digits of Lam,
// `dga`: of |Lam| (the own-outage NaN counts as zero).
__global__ __launch_bounds__(256) void kn_pack(DevNet net, int8_t* __restrict__ dig, int8_t* __restrict__ dga) {
  const int lane = threadIdx.x & 63;
  const int LC = net.Lp / 32;
  const int lc = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (lc >= LC) return;
  const int kt = blockIdx.y;
  const int k = kt * 32 + (lane & 31);
  const int l0 = lc * 32 + 16 * (lane >> 5);
  int s[kLinDigits][4] = {}, a[kLinDigits][4] = {};
  for (int j = 0; j < 16; ++j) {
    float x = k < net.K ? net.lodf[(size_t)k * net.Lp + l0 + j] : 0.0f;
    if (!(fabsf(x) < kLinMaxFactor)) x = 0.0f;
    long long q = (long long)rint((double)x * 0x1p38), m = q < 0 ? -q : q;
#pragma unroll
    for (int d = 0; d < kLinDigits; ++d) {
      const int y = (int)((q + 128) & 255) - 128, z = (int)((m + 128) & 255) - 128;
      q = (q - y) >> 8;
      m = (m - z) >> 8;
      s[d][j / 4] |= (y & 255) << (8 * (j & 3));
      a[d][j / 4] |= (z & 255) << (8 * (j & 3));
    }
  }
  const size_t base = (((size_t)kt * LC + lc) * kLinDigits * 64 + lane) * 16;
#pragma unroll
  for (int d = 0; d < kLinDigits; ++d) {
    *reinterpret_cast<int4*>(dig + base + (size_t)d * 1024) = make_int4(s[d][0], s[d][1], s[d][2], s[d][3]);
    *reinterpret_cast<int4*>(dga + base + (size_t)d * 1024) = make_int4(a[d][0], a[d][1], a[d][2], a[d][3]);
  }
}

// |Lam| of 64 outages spread over each line's row (0 for its own outage and on padding lines).
__global__ __launch_bounds__(256) void kn_sample(DevNet net, float* __restrict__ smp) {
  const int lane = threadIdx.x & 63, l = blockIdx.x * 4 + (threadIdx.x >> 6);
  const float x = l < net.L ? fabsf(net.lodfT[(size_t)l * net.Kp + lin_sample(net.K, lane)]) : 0.0f;
  smp[(size_t)l * 64 + lane] = x < kLinMaxFactor ? x : 0.0f;
}

hipError_t launch_lin_pack(const DevNet& net, int8_t* dig, int8_t* dga, float* smp, hipStream_t s) {
  hipLaunchKernelGGL(kn_sample, dim3(net.Lp / 4), dim3(256), 0, s, net, smp);
  hipLaunchKernelGGL(kn_pack, dim3((net.Lp / 32 + 3) / 4, lin_ktiles(net.K)), dim3(256), 0, s, net, dig, dga);
  return hipGetLastError();
}

// KN1: 64 outages x 64 boxes per block, transposed through LDS.
__global__ __launch_bounds__(256) void kn_outages(DevNet net, void* ws, WsLayout lay, int64_t n_box) {
  __shared__ float2 t[64][65];
  __shared__ float wm[4][64], rm[4][64];
  __shared__ float fk[64];
  __shared__ unsigned wn[4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int k0 = blockIdx.x * 64;
  const int64_t g = blockIdx.y, b0 = g * kLinGroup;
  const int k = k0 + lane;
  if (tid < 64) fk[tid] = k < net.K ? net.fmax_c32[net.ctg_line[k]] : FLT_MAX;
  for (int i = w; i < 64; i += 4) {
    float2 v = make_float2(0.0f, 0.0f);
    if (b0 + i < n_box && k < net.K) {
      const int4 d = ws_ptr<int4>(ws, lay.ctg)[(b0 + i) * net.K + k];
      v = make_float2(__int_as_float(d.y), __int_as_float(d.z));
    }
    t[lane][i] = v;
  }
  __syncthreads();
  float2* oc = ws_ptr<float2>(ws, lay.oc);
  float m = 0.0f, r = 0.0f;
  unsigned wide = 0u;
  for (int i = w; i < 64; i += 4) {
    const float2 v = t[i][lane];
    r = fmaxf(r, v.y);
    wide += v.y > fk[i];
    if (k0 + i < net.K) oc[((size_t)g * net.K + k0 + i) * kLinGroup + lane] = v;
    m = fmaxf(m, fabsf(v.x) + v.y);
  }
  wm[w][lane] = m;
  rm[w][lane] = r;
  wn[w][lane] = wide;
  // per outage the group's largest, raised for the test's float32 roundings
  if (tid < 64) {
    float x = 0.0f;
#pragma unroll 8
    for (int i = 0; i < 64; ++i) {
      const float2 v = t[tid][i];
      x = fmaxf(x, fabsf(v.x) + v.y);
    }
    ws_ptr<float>(ws, lay.ow)[(size_t)g * net.Kp + k0 + tid] = x * (1.0f + 0x1p-20f);
  }
  __syncthreads();
  if (w == 0 && b0 + lane < n_box) {
    m = fmaxf(fmaxf(wm[0][lane], wm[1][lane]), fmaxf(wm[2][lane], wm[3][lane]));
    r = fmaxf(fmaxf(rm[0][lane], rm[1][lane]), fmaxf(rm[2][lane], rm[3][lane]));
    unsigned* slot = reinterpret_cast<unsigned*>(ws_ptr<double>(ws, lay.box) + (b0 + lane) * kBoxSlots + kWmax);
    atomicMax(slot, __float_as_uint(m));
    atomicMax(slot + 1, __float_as_uint(r));
    atomicAdd(slot + 1 - 2 * kWmax, wn[0][lane] + wn[1][lane] + wn[2][lane] + wn[3][lane]);
  }
}

// KN2.  A lane is a box; the lines' factors are scanned 64 outages at a time, a
// lane an outage, against the group's margins, and every element that passes is
// evaluated for all 64 boxes.  Two kinds of (line, box) pairs leave the linear
// model (a = 0) instead, and are swept densely with the dense sweep's own
// float32 elements:
//  - pairs so close to a kink that more than about 5% of the outages could move
//    them across it (KN2p, lanes are outages).  One such box would make its 63
//    neighbours' elements candidates too: 1.4% of the pairs of 2000-bus sub-boxes
//    taken out leave 1.5% of the elements as candidates instead of 7.8%.
//  - quads of lines of which one carries over kHeavy times its limit or, in a wide
//    box (an outaged line's radius over its limit for a third of them), is active on
//    the lower side (KN2h).  Their float32 units are the coarsest, so that almost
//    all of the difference between this sweep and the dense one (which rounds its
//    elements and sums) comes from a few of them; swept like there, both sweeps'
//    bounds agreed to 1e-9 (measured, not assured: 65 networks of 1000 to 8300 buses,
//    sub-boxes, periods and whole boxes; points of zero width at 1500 buses 1.3e-9; every
//    line's limit on its flow 2.6e-6 of a small bound).  18432 boxes at 2000 buses: 3.1 ms (kHeavy = 3: 4.7, 2: 9.9).
// Blocks of one group of boxes run on one XCD, whose L2 then holds the group's
// (c_k, r_k) (1.5 MB at 2954 outages).  Loads and the float64 evaluations of the
// candidates bound it together: four waves per SIMD (128 registers) take 4.0 ms for
// 18432 boxes at 2000 buses, three (134 registers) 5.0, five (spills) 5.2.
constexpr float kHeavy = 4.0f;
constexpr float kTinyRadius = 0x1p-5f;  // of the smallest limit
constexpr int kList = 60;  // candidates of a line listed before they are evaluated
constexpr int kNearRank = 4;  // of 64 sampled outages: the pair threshold is the 4th largest |Lam| w

template <int SIDES>
__global__ __launch_bounds__(256, 4) void kn_lines(DevNet net, void* ws, WsLayout lay, int64_t n_box, int n_lb,
                                                int n_units) {
  constexpr bool UP = SIDES & 2, LO = SIDES & 1;
  __shared__ __align__(16) union {
    float t[(UP + LO + 1) * kLinLines][65];
    int list[4][8][kList + 132];
  } sm;
  __shared__ __align__(16) double red[4 * 4 * 64];
  float (*sc)[65] = sm.t, (*sh)[65] = sm.t + kLinLines, (*sg)[65] = sm.t + (UP + 1) * kLinLines;
  auto& list = sm.list;  // candidate outages per line
  const int per = (n_units + 7) / 8;
  const int u = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || u >= n_units) return;  // the whole block
  const int lb = u % n_lb;
  const int64_t g = u / n_lb, b0 = g * kLinGroup;
  const int l0 = lb * kLinLines;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // the tile's line data, as the dense sweep forms it, transposed into LDS
  {
    const int r = tid >> 3, l4 = (tid & 7) * 4;
    const float4 e4 = *reinterpret_cast<const float4*>(net.line_eps + l0 + l4);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int i = r + 32 * p;
      const int64_t b = b0 + i;
      float4 c = make_float4(0.f, 0.f, 0.f, 0.f), h = make_float4(-FLT_MAX, -FLT_MAX, -FLT_MAX, -FLT_MAX);
      float4 q = make_float4(FLT_MAX, FLT_MAX, FLT_MAX, FLT_MAX);
      if (b < n_box) {
        const double* bs = ws_ptr<double>(ws, lay.box) + b * kBoxSlots;
        const float vmax = __uint_as_float(*reinterpret_cast<const unsigned*>(bs + kVmax));
        const float ex = next_up_f32(e4.x * vmax), ey = next_up_f32(e4.y * vmax);
        const float ez = next_up_f32(e4.z * vmax), ew = next_up_f32(e4.w * vmax);
        const size_t at = (size_t)b * net.Lp + l0 + l4;
        c = *reinterpret_cast<const float4*>(ws_ptr<float>(ws, lay.lc) + at);
        if (UP) {
          h = *reinterpret_cast<const float4*>(ws_ptr<float>(ws, lay.lh) + at);
          h = make_float4(add_ru(h.x, ex), add_ru(h.y, ey), add_ru(h.z, ez), add_ru(h.w, ew));
        }
        if (LO) {
          q = *reinterpret_cast<const float4*>(ws_ptr<float>(ws, lay.lg) + at);
          q = make_float4(add_ru(q.x, ex), add_ru(q.y, ey), add_ru(q.z, ez), add_ru(q.w, ew));
        }
      }
      sc[l4 + 0][i] = c.x; sc[l4 + 1][i] = c.y; sc[l4 + 2][i] = c.z; sc[l4 + 3][i] = c.w;
      if (UP) {
        sh[l4 + 0][i] = h.x; sh[l4 + 1][i] = h.y; sh[l4 + 2][i] = h.z; sh[l4 + 3][i] = h.w;
      }
      if (LO) {
        sg[l4 + 0][i] = q.x; sg[l4 + 1][i] = q.y; sg[l4 + 2][i] = q.z; sg[l4 + 3][i] = q.w;
      }
    }
  }
  __syncthreads();

  // a, v, the lines' own sums and the group's margins: wave w takes lines 8 w ..+7
  // and keeps its boxes' data of them in registers
  double acc_hi = 0.0, acc_lo = 0.0, e_hi = 0.0, e_lo = 0.0;
  int8_t* vb = reinterpret_cast<int8_t*>(red);  // [2 sides][64 boxes][32 lines]
  const float* W = ws_ptr<float>(ws, lay.ow) + (size_t)g * net.Kp;
  float c[8], h[8], q[8], mg[8];
  unsigned lin = 0u;  // bit j: line j of this box is in the model
  {
    const bool in = b0 + lane < n_box;
    const float wk = W[lin_sample(net.K, lane)];
    const float* bs = reinterpret_cast<const float*>(ws_ptr<double>(ws, lay.box) + min(b0 + lane, n_box - 1) * kBoxSlots + kWmax);
    const float wmax = bs[0], rmax = bs[1];
    const bool wide = 3u * __float_as_uint(bs[1 - 2 * kWmax]) > (unsigned)net.K;
    unsigned vu[2] = {0u, 0u}, vl[2] = {0u, 0u};
    uint64_t heavy = 0;
    double th_hi = 0.0, th_lo = 0.0;
    bool all_hi = true, all_lo = true;
    float px0 = 0.0f, px2 = 0.0f, py0 = 0.0f, py2 = 0.0f, mv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = w * 8 + j;
      mv[j] = net.lin_smp[(size_t)(l0 + i) * 64 + lane];
      c[j] = sc[i][lane];
      h[j] = UP ? sh[UP ? i : 0][lane] : 0.0f;
      q[j] = LO ? sg[LO ? i : 0][lane] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int l = l0 + w * 8 + j;
      if ((j & 3) == 0) {
        bool hv = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float f = net.fmax_c32[l + e];
          hv |= fabsf(c[j + e]) > kHeavy * f;
          if (LO) hv |= wide && fabsf(c[j + e]) > q[j + e];
        }
        heavy = __builtin_amdgcn_ballot_w64(hv && in);
        if (lane == 0) ws_ptr<uint64_t>(ws, lay.hq)[(size_t)g * (net.Lp / 4) + l / 4] = heavy;
      }
      // the sampled outages' largest moves of the line's flow
      float m0 = mv[j] * wk;
      m0 = m0 > 0.0f ? m0 : 0.0f;
      unsigned th = 0u;
#pragma unroll
      for (int r = 0; r < kNearRank; ++r) {
        th = wave_max_u32(__float_as_uint(m0));
        if (__float_as_uint(m0) >= th) m0 = 0.0f;
      }
      const float theta = __uint_as_float(th);
      const float ac = fabsf(c[j]);
      float x = 0.0f, y = 0.0f, m = FLT_MAX;
      if (UP) {
        x = ac + h[j];
        m = x > 0.0f ? fminf(x, ac) : -x;
      }
      if (LO) {
        y = ac - q[j];
        m = fminf(m, fabsf(y));
      }
      m = m >= 0.0f ? m : FLT_MAX;  // an invalid box
      const bool hv = (heavy >> lane) & 1;
      const bool near = in && !hv && m < theta && l < net.L;
      const uint64_t nm = __builtin_amdgcn_ballot_w64(near);
      if (lane == 0) ws_ptr<uint64_t>(ws, lay.nk)[(size_t)g * net.Lp + l] = nm;
      const bool on = !hv && !near;
      lin |= (on ? 1u : 0u) << j;
      const bool own = l < net.L && net.ctg_of_line[l] >= 0;  // the line's own outage has no element of it
      const double n = l < net.L ? (double)(net.K - own) : 0.0;
      const unsigned sgn = c[j] < 0.0f ? 0xffu : 1u;
      // A line that no other outage moves (a bridge, or a line of a loop of which no
      // other line is studied) has the same float32 element x or y for all of them in
      // the dense sweep: its rounding is taken as it is there, and so is that of a
      // quad's sum, where every active line of it is such a line and a bridge (n = K).
      const bool rigid = net.lam_max[l] * wmax < 0x1p-26f * ac;
      if ((j & 3) == 0) {
        th_hi = th_lo = 0.0;
        all_hi = all_lo = true;
      }
      float px = 0.0f, py = 0.0f;
      if (UP && on && x > 0.0f) {
        px = x;
        th_hi += n * (rigid ? (double)x : (double)ac + (double)h[j]);
        e_hi += n * ((double)ac + fabs((double)h[j]));
        vu[j >> 2] |= sgn << (8 * (j & 3));
        all_hi &= rigid && !own;
      }
      if (LO && on && y > 0.0f) {
        py = y;
        th_lo += n * (rigid ? (double)y : (double)ac - (double)q[j]);
        e_lo += n * ((double)ac + (double)q[j]);
        vl[j >> 2] |= sgn << (8 * (j & 3));
        all_lo &= rigid && !own;
      }
      // the dense sweep's order: (l0 + l1) + (l2 + l3)
      if (j & 1) {
        (j & 2 ? px2 : px0) += px;
        (j & 2 ? py2 : py0) += py;
      } else {
        (j & 2 ? px2 : px0) = px;
        (j & 2 ? py2 : py0) = py;
      }
      if ((j & 3) == 3) {
        acc_hi += all_hi ? (double)net.K * (double)(px0 + px2) : th_hi;
        acc_lo += all_lo ? (double)net.K * (double)(py0 + py2) : th_lo;
      }
      // the smallest margin of the boxes in the model, lowered for the test's float32 roundings
      const unsigned mb = 0x7f800000u - __float_as_uint(on ? m : FLT_MAX);
      mg[j] = __uint_as_float(0x7f800000u - wave_max_u32(mb)) * (1.0f - 0x1p-20f);
    }
    // In boxes of next to no width |Lam| r_k mostly lies below half a unit of h (of
    // g), and the dense sweep's float32 A (B) loses it: 3e-10 of the penalties at
    // 2000 buses, 1e-9 at 1000.  The same amount, estimated from the sampled
    // outages, is left out here.  The estimate need not be right: e holds, in full, what
    // it moves the total by (the finalize multiplies e by the factor in `charge`).
    const float tiny = kTinyRadius * (float)net.fmax_c_min;
    if (__builtin_amdgcn_ballot_w64(in && rmax < tiny) != 0) {
      double uh[8] = {}, ul[8] = {};
      const float2* oq = ws_ptr<float2>(ws, lay.oc) + (size_t)g * net.K * kLinGroup + lane;
      const float* smp = net.lin_smp + (size_t)(l0 + w * 8) * 64;
      for (int t = 0; t < 64; ++t) {
        const float rk = oq[(size_t)lin_sample(net.K, t) * kLinGroup].y;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float z = smp[j * 64 + t];
          if (UP) uh[j] += (double)fmaf(-z, rk, fmaf(z, rk, h[j]) - h[j]);
          if (LO) ul[j] += (double)fmaf(-z, rk, fmaf(z, rk, q[j]) - q[j]);
        }
      }
      const double per = rmax < tiny ? (double)net.K / 64.0 : 0.0;
      const double charge = 1.0 / (4.0 * (double)(net.L + net.K + 4096) * kU64);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (UP && ((vu[j >> 2] >> (8 * (j & 3))) & 1)) {
          acc_hi += per * uh[j];
          e_hi += charge * per * fabs(uh[j]);
        }
        if (LO && ((vl[j >> 2] >> (8 * (j & 3))) & 1)) {
          acc_lo -= per * ul[j];
          e_lo += charge * per * fabs(ul[j]);
        }
      }
    }
    if (UP) *reinterpret_cast<uint2*>(vb + lane * 32 + w * 8) = make_uint2(vu[0], vu[1]);
    if (LO) *reinterpret_cast<uint2*>(vb + 2048 + lane * 32 + w * 8) = make_uint2(vl[0], vl[1]);
  }
  __syncthreads();
  {
    // operand order of the products: [32 boxes][32 lines][64 lanes][16 bytes]
    const int side = tid >> 7, bt = (tid >> 6) & 1;
    if ((side == 0 && UP) || (side == 1 && LO)) {
      const int4 v = *reinterpret_cast<const int4*>(vb + side * 2048 + (bt * 32 + (lane & 31)) * 32 + 16 * (lane >> 5));
      int8_t* vf = ws_ptr<int8_t>(ws, side == 0 ? lay.vu : lay.vl);
      *reinterpret_cast<int4*>(vf + (((size_t)(g * 2 + bt) * n_lb + lb) * 64 + lane) * 16) = v;
    }
  }

  // exceptions: wave w scans its 8 lines' factors, lists each line's candidates and
  // evaluates the lists.  With s = sign(c_l), D = |C| - s C and X = |C| + A the true
  // penalty minus the linear one is max(-X, 0) + D where the side is active at the
  // base flow, max(X, 0) where not (lower side: X = |C| - B); D is summed once for
  // both sides.  A zero factor gives exactly zero and fills the last group of four.
  const char* oc = reinterpret_cast<const char*>(ws_ptr<float2>(ws, lay.oc) + (size_t)g * net.K * kLinGroup);
  const unsigned lane8 = lane * 8u;
  const int n_kc = (net.K + 63) / 64;
  int (*lst)[kList + 132] = list[w];  // in the memory of the tile, which every wave has read by now
  const float* lp[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) lp[j] = net.lodfT + (size_t)min(l0 + w * 8 + j, net.L - 1) * net.Kp;
  int cnt[8] = {};
  // the next 64 outages' factors are loaded while these are tested
  float ln[8], wn = W[lane];
#pragma unroll
  for (int j = 0; j < 8; ++j) ln[j] = lp[j][lane];
  for (int kc = 0;; ++kc) {
    const bool last = kc >= n_kc;
    if (!last) {
      const int k = kc * 64 + lane, kn = min(kc + 1, n_kc - 1) * 64 + lane;
      const float wk = wn;
      float la[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) la[j] = ln[j];
      wn = W[kn];
#pragma unroll
      for (int j = 0; j < 8; ++j) ln[j] = lp[j][kn];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // (a line's own outage is NaN: false)
        const uint64_t mask = __builtin_amdgcn_ballot_w64(fabsf(lin_factor(la[j])) * wk > mg[j]);
        if (mask == 0) continue;
        const int rank =
            __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
        if ((mask >> lane) & 1) lst[j][cnt[j] + rank] = k;
        cnt[j] = __builtin_amdgcn_readfirstlane(cnt[j] + __builtin_popcountll(mask));
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (cnt[j] <= (last ? 0 : kList)) continue;
      const double cd = c[j], hd = h[j], qd = q[j];
      const bool au = fabsf(c[j]) + h[j] > 0.0f, al = fabsf(c[j]) - q[j] > 0.0f;
      const unsigned cs = __float_as_uint(c[j]) & 0x80000000u, us = au ? 0x80000000u : 0u, ls = al ? 0x80000000u : 0u;
      double dh = 0.0, dl = 0.0, dd = 0.0;
      if (lane < 3) lst[j][cnt[j] + lane] = -1;
      for (int t = 0; t < cnt[j]; t += 4) {
        const int4 k4 = *reinterpret_cast<const int4*>(&lst[j][t]);
        const int ks[4] = {k4.x, k4.y, k4.z, k4.w};
        float lam[4];
        float2 o[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const unsigned k = (unsigned)max(ks[r], 0);
          lam[r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(lp[j]) + k * 4u);
          o[r] = *reinterpret_cast<const float2*>(oc + (k * (kLinGroup * 8u) + lane8));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double lm = ks[r] >= 0 ? lin_factor(lam[r]) : 0.0f, rk = o[r].y;
          const double C = fma(lm, (double)o[r].x, cd);
          dd += relu_neg(flip_sign(C, cs));
          if (UP) dh += relu(flip_sign(fabs(C) + fma(fabs(lm), rk, hd), us));
          if (LO) dl += relu(flip_sign(fabs(C) - fma(fabs(lm), rk, qd), ls));
        }
      }
      cnt[j] = 0;
      // pairs out of the model are summed elsewhere
      const bool on = (lin >> j) & 1;
      if (UP) acc_hi += on ? dh + (au ? 2.0 * dd : 0.0) : 0.0;
      if (LO) acc_lo += on ? dl + (al ? 2.0 * dd : 0.0) : 0.0;
    }
    if (last) break;
  }

  // per box: the four waves' sums in order
  __syncthreads();
  red[(0 * 4 + w) * 64 + lane] = acc_hi;
  red[(1 * 4 + w) * 64 + lane] = acc_lo;
  red[(2 * 4 + w) * 64 + lane] = e_hi;
  red[(3 * 4 + w) * 64 + lane] = e_lo;
  __syncthreads();
  if (w < 2 && b0 + lane < n_box) {
    const double* r = red + w * 8 * 64 + lane;
    const double x = (r[0] + r[64]) + (r[128] + r[192]), y = (r[256] + r[320]) + (r[384] + r[448]);
    const int64_t b = b0 + lane;
    if (w == 0)
      ws_ptr<double2>(ws, lay.p3)[b * lay.n_p3 + lb] = make_double2(x, y);
    else
      ws_ptr<double2>(ws, lay.pe)[b * lay.n_pe + lb] = make_double2(x, y);
  }
}

// KN2p: the pairs near a kink.  A block takes one box and 2048 outages (eight per
// lane, kept in registers) and walks the box's marked lines, the next line's data loaded
// ahead.  A line's own steps (its padded limits) and a wait per line bound it: 18432 boxes at
// 2000 buses 1.55 ms with four outages per lane and no load ahead, 1.38 with the load, 1.1
// with eight.
constexpr int kPairQ = 8;
constexpr int kPairChunk = 256 * kPairQ;  // (lin_pair_chunks)
constexpr int kPairSeg = 2048;  // lines listed in LDS at a time

template <int SIDES>
__global__ __launch_bounds__(256) void kn_pairs(DevNet net, void* ws, WsLayout lay, int64_t box0, int slot0) {
  __shared__ int list[kPairSeg];
  __shared__ int cnt[4];
  __shared__ double red[8];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = box0 + blockIdx.x;
  const int64_t g = b / kLinGroup;
  const int bit = (int)(b % kLinGroup);
  const double* bs = ws_ptr<double>(ws, lay.box) + b * kBoxSlots;
  const float vmax = __uint_as_float(*reinterpret_cast<const unsigned*>(bs + kVmax));
  const int kw = blockIdx.y * kPairChunk + w * 64 * kPairQ + lane;
  float cc[kPairQ], rk[kPairQ];
#pragma unroll
  for (int q = 0; q < kPairQ; ++q) {
    const int k = kw + 64 * q;
    const int4 d = ws_ptr<int4>(ws, lay.ctg)[b * net.K + min(k, net.K - 1)];
    cc[q] = __int_as_float(d.y);
    rk[q] = __int_as_float(d.z);
  }
  const uint64_t* nk = ws_ptr<uint64_t>(ws, lay.nk) + (size_t)g * net.Lp;
  const float* lc = ws_ptr<float>(ws, lay.lc) + b * net.Lp;
  const float* lh = ws_ptr<float>(ws, lay.lh) + b * net.Lp;
  const float* lg = ws_ptr<float>(ws, lay.lg) + b * net.Lp;
  double acc_hi = 0.0, acc_lo = 0.0;
  for (int s0 = 0; s0 < net.Lp; s0 += kPairSeg) {
    // the segment's marked lines in order: wave w takes a quarter of it
    const int per = kPairSeg / 4;
    const int base = s0 + w * per;
    int n = 0;
    for (int j = 0; j < per; j += 64) {
      const int l = base + j + lane;
      const bool on = l < net.Lp && ((nk[min(l, net.Lp - 1)] >> bit) & 1);
      const uint64_t m = __builtin_amdgcn_ballot_w64(on);
      const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      if (on) list[w * per + n + rank] = l;
      n += __builtin_popcountll(m);
    }
    if (lane == 0) cnt[w] = n;
    __syncthreads();
    // the marked lines in order, each one's data loaded while the line before it is summed
    int v = 0, j = 0;
    auto settle = [&] {
      while (v < 4 && j >= cnt[v]) {
        ++v;
        j = 0;
      }
      return v < 4;
    };
    float4 d;  // (c, h, g, line_eps) as stored
    float x[kPairQ];
    auto load = [&] {
      const int l = __builtin_amdgcn_readfirstlane(list[v * per + j]);
      d = make_float4(lc[l], lh[l], lg[l], net.line_eps[l]);
      const float* row = net.lodfT + (size_t)l * net.Kp;
#pragma unroll
      for (int e = 0; e < kPairQ; ++e) x[e] = row[min(kw + 64 * e, net.K - 1)];
    };
    bool more = kw - lane < net.K && settle();  // (no outage left for this wave)
    if (more) load();
    while (more) {
      const float4 t = d;
      float lam[kPairQ];
#pragma unroll
      for (int e = 0; e < kPairQ; ++e) lam[e] = x[e];
      ++j;
      more = settle();
      if (more) load();
      const float ex = next_up_f32(t.w * vmax);
      const float h = add_ru(t.y, ex), q = add_ru(t.z, ex);
      float p[kPairQ], r[kPairQ];
#pragma unroll
      for (int e = 0; e < kPairQ; ++e) {
        k3_elem<SIDES>(lam[e], cc[e], rk[e], t.x, h, q, p[e], r[e]);
        if (kw + 64 * e >= net.K) p[e] = r[e] = 0.0f;
      }
      // float32 sums of four outages
#pragma unroll
      for (int e = 0; e < kPairQ; e += 4) {
        if (SIDES & 2) acc_hi += (double)((p[e] + p[e + 1]) + (p[e + 2] + p[e + 3]));
        if (SIDES & 1) acc_lo += (double)((r[e] + r[e + 1]) + (r[e + 2] + r[e + 3]));
      }
    }
    __syncthreads();
  }
  acc_hi = wave_sum(acc_hi);
  acc_lo = wave_sum(acc_lo);
  if (lane == 0) {
    red[w] = acc_hi;
    red[4 + w] = acc_lo;
  }
  __syncthreads();
  if (tid == 0)
    ws_ptr<double2>(ws, lay.p3)[b * lay.n_p3 + slot0 + blockIdx.y] =
        make_double2((red[0] + red[1]) + (red[2] + red[3]), (red[4] + red[5]) + (red[6] + red[7]));
}

// KN2h: the heavy quads, a lane a box: kHeavyLines lines x kHeavyK outages per
// block, a quarter of the outages per wave.  Factors are wave-uniform (scalar
// loads, one copy into a vector register each), (c_k, r_k) one coalesced row per
// outage; elements and float32 sums (four lines x two outages) are the dense sweep's.

template <int SIDES>
__global__ __launch_bounds__(256) void kn_heavy(DevNet net, void* ws, WsLayout lay, int64_t n_box, int slot0) {
  constexpr bool UP = SIDES & 2, LO = SIDES & 1;
  __shared__ double red[2 * 4 * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t g = blockIdx.y, b = g * kLinGroup + lane;
  const int64_t bq = min(b, n_box - 1);
  const int q0 = blockIdx.x * (kHeavyLines / 4), q1 = min(q0 + kHeavyLines / 4, net.Lp / 4);
  const int k0 = blockIdx.z * kHeavyK + w * (kHeavyK / 4), k1 = min(k0 + kHeavyK / 4, net.K);
  const float2* oc = ws_ptr<float2>(ws, lay.oc) + (size_t)g * net.K * kLinGroup + lane;
  const uint64_t* hqs = ws_ptr<uint64_t>(ws, lay.hq) + (size_t)g * (net.Lp / 4);
  const double* bs = ws_ptr<double>(ws, lay.box) + bq * kBoxSlots;
  const float vmax = __uint_as_float(*reinterpret_cast<const unsigned*>(bs + kVmax));
  typedef __attribute__((address_space(4))) const float const_float;
  double acc_hi = 0.0, acc_lo = 0.0;
  for (int t = q0; t < q1; ++t) {
    const uint64_t hq = hqs[t];
    if (hq == 0) continue;
    const float4 e4 = reinterpret_cast<const float4*>(net.line_eps)[t];
    const float ex = next_up_f32(e4.x * vmax), ey = next_up_f32(e4.y * vmax);
    const float ez = next_up_f32(e4.z * vmax), ew = next_up_f32(e4.w * vmax);
    const size_t at = (size_t)bq * net.Lp + 4 * t;
    const float4 c = *reinterpret_cast<const float4*>(ws_ptr<float>(ws, lay.lc) + at);
    float4 h = make_float4(0.f, 0.f, 0.f, 0.f), q = h;
    if (UP) {
      h = *reinterpret_cast<const float4*>(ws_ptr<float>(ws, lay.lh) + at);
      h = make_float4(add_ru(h.x, ex), add_ru(h.y, ey), add_ru(h.z, ez), add_ru(h.w, ew));
    }
    if (LO) {
      q = *reinterpret_cast<const float4*>(ws_ptr<float>(ws, lay.lg) + at);
      q = make_float4(add_ru(q.x, ex), add_ru(q.y, ey), add_ru(q.z, ez), add_ru(q.w, ew));
    }
    const_float* lr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) lr[i] = (const_float*)(net.lodfT + (size_t)min(4 * t + i, net.L - 1) * net.Kp);
    double dh = 0.0, dl = 0.0;
    auto two = [&](const float4& x0, const float2& o0, const float4& x1, const float2& o1) {
      k3_pair<SIDES>(x0, make_int4(0, __float_as_int(o0.x), __float_as_int(o0.y), 0), x1,
                     make_int4(0, __float_as_int(o1.x), __float_as_int(o1.y), 0), c, h, q, dh, dl);
    };
    int k = k0;
    for (; k + 8 <= k1; k += 8) {
      float2 o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = oc[(size_t)(k + e) * kLinGroup];
      float4 x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = make_float4(lr[0][k + e], lr[1][k + e], lr[2][k + e], lr[3][k + e]);
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const float4 a = make_float4(vcopy(x[e].x), vcopy(x[e].y), vcopy(x[e].z), vcopy(x[e].w));
        const float4 d = make_float4(vcopy(x[e + 1].x), vcopy(x[e + 1].y), vcopy(x[e + 1].z), vcopy(x[e + 1].w));
        two(a, o[e], d, o[e + 1]);
      }
    }
    for (; k < k1; k += 2) {
      // an odd last outage is paired with itself at r = NaN, whose penalties are 0
      const bool on = k + 1 < k1;
      const int kb = on ? k + 1 : k;
      const float2 oa = oc[(size_t)k * kLinGroup];
      float2 ob = oc[(size_t)kb * kLinGroup];
      if (!on) ob.y = NAN;
      two(make_float4(lr[0][k], lr[1][k], lr[2][k], lr[3][k]), oa,
          make_float4(lr[0][kb], lr[1][kb], lr[2][kb], lr[3][kb]), ob);
    }
    const bool hv = (hq >> lane) & 1;
    acc_hi += hv ? dh : 0.0;
    acc_lo += hv ? dl : 0.0;
  }
  red[w * 64 + lane] = acc_hi;
  red[256 + w * 64 + lane] = acc_lo;
  __syncthreads();
  if (w == 0 && b < n_box) {
    const double* r = red + lane;
    ws_ptr<double2>(ws, lay.p3)[b * lay.n_p3 + slot0 + blockIdx.x * gridDim.z + blockIdx.z] =
        make_double2((r[0] + r[64]) + (r[128] + r[192]), (r[256] + r[320]) + (r[384] + r[448]));
  }
}

// KN3: one wave takes 32 outages (five digit planes) x 64 boxes, a block MW x NW
// waves.  Operands are staged through LDS two 32-line steps at a time, the next
// pair loaded into registers while this one is multiplied (160 accumulator
// registers, two waves per SIMD).  Pass z: side (upper, lower) x (signed with v,
// absolute with a = v & 1).  The digit sums are joined and weighted in float64
// per (box, 32 outages).
template <int MW, int NW>
__global__ __launch_bounds__(64 * MW * NW) void kn_gemm(DevNet net, void* ws, WsLayout lay, int64_t n_box,
                                                        int n_lc, int n_kt, int n_mb, int n_nb, int side0) {
  constexpr int kWaves = MW * NW;
  constexpr int kA = MW * 2 * kLinDigits, kUnits = kA + NW * 4;  // 1 KB units of a stage
  constexpr int kPer = (kUnits + kWaves - 1) / kWaves;
  __shared__ __align__(16) int8_t stage[2 * kUnits * 1024];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mw = w % MW, nw = w / MW;
  // blocks of one XCD on consecutive tiles, outage blocks fastest: they share the boxes' operand
  const int n_units = n_mb * n_nb, per = (n_units + 7) / 8;
  const int u = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || u >= n_units) return;  // the whole block
  const int kt0 = (u % n_mb) * MW, bt0 = (u / n_mb) * NW * 2;
  const int side = side0 + (blockIdx.y >> 1), abs_ = blockIdx.y & 1;
  const int n_bt = (int)((n_box + kLinGroup - 1) / kLinGroup) * 2;
  const int8_t* A = abs_ ? net.lin_dga : net.lin_dig;
  const int8_t* V = ws_ptr<int8_t>(ws, side == 0 ? lay.vu : lay.vl);
  const int8_t* src[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int q = min(w + i * kWaves, kUnits - 1);
    if (q < kA) {
      const int m = q / (2 * kLinDigits), off = q % (2 * kLinDigits);
      src[i] = A + (size_t)min(kt0 + m, n_kt - 1) * n_lc * (kLinDigits * 1024) + off * 1024 + lane * 16;
    } else {
      const int n = (q - kA) / 2, off = (q - kA) % 2;
      src[i] = V + (size_t)min(bt0 + n, n_bt - 1) * n_lc * 1024 + off * 1024 + lane * 16;
    }
  }
  v16i acc[kLinDigits][2];
#pragma unroll
  for (int d = 0; d < kLinDigits; ++d)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[d][j][r] = 0;
  const int n_st = n_lc / 2;
  v4i pre[kPer];
  auto fetch = [&](int s) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int step = w + i * kWaves < kA ? 2 * kLinDigits * 1024 : 2 * 1024;  // wave-uniform
      pre[i] = *reinterpret_cast<const v4i*>(src[i] + (size_t)s * step);
    }
  };
  auto put = [&](int s) {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (w + i * kWaves < kUnits)
        *reinterpret_cast<v4i*>(stage + ((s & 1) * kUnits + w + i * kWaves) * 1024 + lane * 16) = pre[i];
  };
  fetch(0);
  put(0);
  __syncthreads();
  const int vmask = abs_ ? 0x01010101 : -1;
  for (int s = 0; s < n_st; ++s) {
    if (s + 1 < n_st) fetch(s + 1);
    const int8_t* st = stage + (s & 1) * kUnits * 1024 + lane * 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v4i b[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        b[j] = *reinterpret_cast<const v4i*>(st + (kA + (nw * 2 + j) * 2 + h) * 1024);
        b[j] = b[j] & vmask;
      }
#pragma unroll
      for (int d = 0; d < kLinDigits; ++d) {
        const v4i a = *reinterpret_cast<const v4i*>(st + (mw * 2 * kLinDigits + h * kLinDigits + d) * 1024);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[d][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[j], acc[d][j], 0, 0, 0);
      }
    }
    if (s + 1 < n_st) put(s + 1);
    __syncthreads();
  }
  const int kt = kt0 + mw;
  if (kt >= n_kt) return;
  // element r of lane t: outage 8 (r / 4) + 4 (t / 32) + r % 4 of the 32, box t % 32
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int bt = bt0 + nw * 2 + j;
    if (bt >= n_bt) break;  // uniform
    const int64_t b = (int64_t)bt * 32 + (lane & 31);
    const float2* oc = ws_ptr<float2>(ws, lay.oc) + (size_t)(bt >> 1) * net.K * kLinGroup + (bt & 1) * 32 + (lane & 31);
    double s = 0.0, e = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int k = kt * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      const float2 o = oc[(size_t)min(k, net.K - 1) * kLinGroup];  // rows past the last outage have zero digits
      // a digit sum is at most 128 L, so two of them join in 32 bits up to kLinMaxLines lines
      const int y01 = acc[1][j][r] * 256 + acc[0][j][r], y23 = acc[3][j][r] * 256 + acc[2][j][r];
      const double y = fma((double)acc[4][j][r], 0x1p-6, fma((double)y23, 0x1p-22, (double)y01 * 0x1p-38));
      if (abs_) {
        s = fma(y, (double)o.y, s);
        e = fma(y, (double)(fabsf(o.x) + o.y), e);
      } else {
        s = fma(y, (double)o.x, s);
      }
    }
    s += __shfl_xor(s, 32, 64);
    e += __shfl_xor(e, 32, 64);
    if (lane < 32 && b < n_box) {
      if (side == 1 && abs_) s = -s;  // |C| - B
      double* p3 = ws_ptr<double>(ws, lay.p3) + (b * lay.n_p3 + lay.lin_lb + abs_ * n_kt + kt) * 2 + side;
      *p3 = s;
      if (abs_) ws_ptr<double>(ws, lay.pe)[(b * lay.n_pe + lay.lin_lb + kt) * 2 + side] = e;
    }
  }
}

template <int MW, int NW>
static hipError_t launch_gemm(const DevNet& net, int64_t n_box, void* ws, const WsLayout& lay, int sides, hipStream_t s) {
  const int n_kt = lin_ktiles(net.K), n_lc = net.Lp / 32;
  const int n_mb = (n_kt + MW - 1) / MW, n_nb = (int)((n_box + kLinGroup * NW - 1) / (kLinGroup * NW));
  const int per = (n_mb * n_nb + 7) / 8;
  hipLaunchKernelGGL((kn_gemm<MW, NW>), dim3(8 * per, sides == 3 ? 4 : 2), dim3(64 * MW * NW), 0, s, net, ws, lay,
                     n_box, n_lc, n_kt, n_mb, n_nb, sides == 1 ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_linear_sweep(const DevNet& net, int64_t n_box, void* ws, const WsLayout& lay, hipStream_t s,
                               KernelTimer* tm) {
  const int64_t G = (n_box + kLinGroup - 1) / kLinGroup;
  int t = tm->start(15, s);
  hipLaunchKernelGGL(kn_outages, dim3((net.K + 63) / 64, (unsigned)G), dim3(256), 0, s, net, ws, lay, n_box);
  const int n_lb = net.Lp / kLinLines, units = (int)(n_lb * G);
  const dim3 grid(8 * ((units + 7) / 8));
  const int slot0 = lay.lin_lb + 2 * lin_ktiles(net.K), slot1 = slot0 + lin_pair_chunks(net.K);
  auto go = [&](auto sides) {
    constexpr int SIDES = decltype(sides)::value;
    hipLaunchKernelGGL(kn_lines<SIDES>, grid, dim3(256), 0, s, net, ws, lay, n_box, n_lb, units);
    for (int64_t b0 = 0; b0 < n_box; b0 += 65535)
      hipLaunchKernelGGL(kn_pairs<SIDES>, dim3((unsigned)std::min<int64_t>(65535, n_box - b0), lin_pair_chunks(net.K)),
                         dim3(256), 0, s, net, ws, lay, b0, slot0);
    hipLaunchKernelGGL(kn_heavy<SIDES>, dim3(lin_heavy_tiles(net.Lp), (unsigned)G, lin_heavy_chunks(net.K)), dim3(256),
                       0, s, net, ws, lay, n_box, slot1);
  };
  if (lay.sides == 1)
    go(std::integral_constant<int, 1>());
  else if (lay.sides == 2)
    go(std::integral_constant<int, 2>());
  else
    go(std::integral_constant<int, 3>());
  tm->stop(t, s);
  t = tm->start(6, s);
  const hipError_t e = n_box > kLinGroup ? launch_gemm<2, 4>(net, n_box, ws, lay, lay.sides, s)
                                         : launch_gemm<4, 1>(net, n_box, ws, lay, lay.sides, s);
  tm->stop(t, s);
  return e;
}

}  // namespace ibp
