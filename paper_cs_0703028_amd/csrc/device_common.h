// device_common.h -- device code shared by the single-case kernels and the
// persistent batched kernel (gfx950): the line-sum tile, Philox ray
// sampling, exact integer traversal, wavefront reductions and the march of
// one wavefront over one spectral chunk of one ray.
#pragma once

#include <type_traits>

#include "rt_internal.h"

namespace rt {
namespace dev {

constexpr int kKappaThreads = 256;
constexpr int kLineTile = 256;
constexpr int kKappaCells = 8;   // cells per lane in the line sum
constexpr int kKappaPoints = 2;  // nu points per lane in the line sum
constexpr int kKappaTilePoints = kKappaThreads * kKappaPoints;
constexpr int kPlainQ = 12;      // the same in the plain form's (kMarchPoints = 64 kPlainQ)

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// e^y for a double argument: range reduction y*log2(e) = n + f in FP64,
// |f| <= 1/2, then 2^f with the hardware base-2 exponential and an exact
// power-of-two scaling.  Error ~1.5e-7 relative over the whole range (the
// FP32 rounding of f contributes < 2.1e-8).
__device__ __forceinline__ float exp_split(double y) {
  double z = y * 1.4426950408889634074;
  double n = rint(z);
  float f = (float)(z - n);
  return ldexpf(fast_exp2(f), (int)n);
}

// 1 - e^{-x} for x >= 0 without cancellation: Taylor series of
// (1 - e^{-x})/x to degree 5 for x < 1/4 (truncation < 5e-8 relative),
// otherwise 1 - e^{-x} (the subtraction loses at most a factor 3.5).
__device__ __forceinline__ float one_minus_exp_neg_d(double x) {
  float xf = (float)x;
  if (xf < 0.25f) {
    float p = fmaf(xf, -1.0f / 720.0f, 1.0f / 120.0f);
    p = fmaf(xf, p, -1.0f / 24.0f);
    p = fmaf(xf, p, 1.0f / 6.0f);
    p = fmaf(xf, p, -0.5f);
    p = fmaf(xf, p, 1.0f);
    return xf * p;
  }
  return 1.0f - exp_split(-x);
}

// ------------------------------------------------- FP32 exponentials (pairs)
// The precision form evaluates every exponential in FP32.  An argument comes
// as an FP32 pair x = h + l (products of pairs keep about 46 bits, so the
// argument's own rounding does not limit the result), e^x is taken by Cody
// and Waite's range reduction with log2(e) split as L_h + L_l:
//   n = rint(h L_h),  f = fma(h, L_h, -n) + (h L_l + l L_h),  e^x = 2^n 2^f,
// |f| <= 1/2 + 2^-20, with the hardware base-2 exponential for 2^f (below
// one ulp) and an exact scaling by 2^n.  Relative error about 1e-7 for
// |x| < 80.
struct Pair {
  float h, l;
};

__device__ __forceinline__ Pair pair_of(float2 v) { return Pair{v.x, v.y}; }

// (a.h + a.l)(b.h + b.l) to about 2^-46 relative: the exact rounding error
// of a.h b.h (one FMA) plus the cross terms; a.l b.l is dropped.
__device__ __forceinline__ Pair pair_mul(Pair a, Pair b) {
  const float p = a.h * b.h;
  const float e = fmaf(a.h, b.l, fmaf(a.l, b.h, fmaf(a.h, b.h, -p)));
  return Pair{p, e};
}

__device__ __forceinline__ float exp_pair(Pair x) {
  constexpr float L_h = 1.44269502162933349609375f;  // log2(e) rounded to FP32
  constexpr float L_l = 1.925962989e-08f;             // log2(e) - L_h
  const float n = rintf(x.h * L_h);
  const float f = fmaf(x.h, L_h, -n) + fmaf(x.h, L_l, x.l * L_h);
  return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// e^x - 1 for x >= 0: below 1/2 the Taylor series to degree 10 (truncation
// below 3e-10 relative) in Horner form, otherwise exp_pair(x) - 1 (the
// subtraction loses at most a factor e^(1/2)/(e^(1/2) - 1) = 2.5).
__device__ __forceinline__ float expm1_pair(Pair x) {
  if (x.h < 0.5f) {
    const float t = x.h + x.l;
    float p = 1.0f + t * (1.0f / 10.0f);
#pragma unroll
    for (int k = 9; k >= 2; --k) p = fmaf(t * (1.0f / (float)k), p, 1.0f);
    return t * p;
  }
  return exp_pair(x) - 1.0f;
}

// 1 - e^{-x} for x >= 0: the alternating series to degree 10 below 1/2,
// otherwise 1 - exp_pair(-x) (loses at most a factor 1/(1 - e^(-1/2)) = 2.5).
__device__ __forceinline__ float one_minus_exp_neg_pair(Pair x) {
  if (x.h < 0.5f) {
    const float t = x.h + x.l;
    float p = 1.0f - t * (1.0f / 10.0f);
#pragma unroll
    for (int k = 9; k >= 2; --k) p = fmaf(-t * (1.0f / (float)k), p, 1.0f);
    return t * p;
  }
  return 1.0f - exp_pair(Pair{-x.h, -x.l});
}

// nu_j = nu0 + j dnu as an FP32 pair, from the pairs of nu0 and dnu: the
// product j dnu.h with its exact rounding error (one FMA), then Knuth's
// TwoSum with nu0.h.
__device__ __forceinline__ Pair nu_at(int64_t j, Pair nu0, Pair dnu) {
  const float jf = (float)j;  // exact below 2^24
  const float ph = jf * dnu.h;
  const float pl = fmaf(jf, dnu.h, -ph) + jf * dnu.l;
  const float s = nu0.h + ph;
  const float bp = s - nu0.h;
  const float err = (nu0.h - (s - bp)) + (ph - bp);
  return Pair{s, err + pl + nu0.l};
}

// Eq. (4) in FP32: B = c1 nu^3 / expm1(theta nu), theta = c2 / T, with the
// argument theta nu formed as a pair product and expm1_pair.
__device__ __forceinline__ float planck_f32(Pair nu, Pair theta, float c1) {
  const float em1 = expm1_pair(pair_mul(nu, theta));
  const float v = nu.h + nu.l;
  return c1 * v * v * v / em1;
}

// Knuth's TwoSum: s + x = s' + err exactly.
__device__ __forceinline__ void two_sum_acc(float& s, float& comp, float x) {
  float t = s + x;
  float bp = t - s;
  float err = (s - (t - bp)) + (x - bp);
  s = t;
  comp += err;
}

// ---------------------------------------------------- wavefront reductions
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_f64(double v) {
  const int2 h = *reinterpret_cast<int2*>(&v);
  int2 r;
  r.x = __builtin_amdgcn_update_dpp(0, h.x, CTRL, ROW_MASK, 0xf, false);
  r.y = __builtin_amdgcn_update_dpp(0, h.y, CTRL, ROW_MASK, 0xf, false);
  return *reinterpret_cast<double*>(&r);
}

// ------------------------------------------------------------ line records
// A staged line: (m, phi, lo, hi) -- the integer centre, the fraction, and
// the first and last offsets from m of the points the line contributes to
// -- then, per cell, (A, g2): the Lorentz amplitude u S s gamma / (pi dnu^2)
// and the squared half width (gamma/dnu)^2 in grid units, so that the line
// adds A / ((j - m - phi)^2 + g2) at point j.
constexpr int kLineRec = 4 + 2 * kKappaCells;  // floats per staged line

// The per-cell part of a record (Eqs. (1)-(2)) from a line's data and a
// cell's factors.
struct CellFactors {
  double beta, theta;
  float G, P, lam2;
};
__device__ __forceinline__ void line_cell_params(const LineData& d, const CellFactors& c,
                                                 int have_E, float& amp, float& g2) {
  const float gp = d.gamma * c.P * fast_exp2(d.nexp * c.lam2);
  float a = c.G * d.S * gp;
  if (have_E) {
    a *= exp_split(d.E2 * c.beta);
    a *= one_minus_exp_neg_d(d.nu * c.theta);
  }
  amp = a;
  g2 = gp * gp;
}
__device__ __forceinline__ void line_cell_params(const LineSet& L, const CellSet& C, int i,
                                                 int64_t cell, int have_E, float& amp, float& g2) {
  line_cell_params(LineData{0.f, 0.f, 0.f, L.S[i], L.gamma[i], L.nexp[i], 0.f, 0.f,
                            have_E ? L.E2[i] : 0.0, have_E ? L.nu[i] : 0.0},
                   CellFactors{C.beta[cell], C.theta[cell], C.G[cell], C.P[cell], C.lam2[cell]},
                   have_E, amp, g2);
}

// The same record in FP32 only (the precision form): the Eq. (1) factors from
// the host-formed FP32 inputs with exp_pair, the half width's temperature
// power and the partition ratio (in Gq) with the hardware base-2 exponential.
struct CellFactors32 {
  float2 beta2, theta2;
  float Gq, Pf, lamf;
};
__device__ __forceinline__ void line_cell_params_f32(const LineSet& L, const CellFactors32& c, int i,
                                                     int have_E, float& amp, float& g2) {
  const float gp = L.gamma[i] * c.Pf * fast_exp2(L.nexp[i] * c.lamf);
  float a = c.Gq * L.S[i] * gp;
  if (have_E) {
    a *= exp_pair(pair_mul(pair_of(L.E2p[i]), pair_of(c.beta2)));
    a *= one_minus_exp_neg_pair(pair_mul(pair_of(L.nup[i]), pair_of(c.theta2)));
  }
  amp = a;
  g2 = gp * gp;
}

// The walls' row B(nu_j, T_wall); theta = c2 / T_wall (zero: cold walls).  Its
// blocks ride in a launch of the same call, behind that launch's own.  A launch
// of its own took 4.5 us, nearly all latency; a plain line sum with it, without:
// 4^3 cells, 1,000 points 28.2, 26.3 us, 5 x 6 x 7 cells, 3,037 points 38.4, 36.4,
// 8^3 cells, 10,000 points, dense 745, 736.
struct WallRow {
  float2 theta, nu0, dnu;
  float c1;
  int n_nu;
  int64_t ld;
  float* out = nullptr;
  unsigned first = 0xffffffffu;  // its first block in the launch
};

__device__ __forceinline__ void wall_row(const WallRow& w, int64_t block, int threads) {
  const int64_t j = block * threads + threadIdx.x;
  if (j >= w.ld) return;
  float v = 0.f;
  if (j < w.n_nu && w.theta.x > 0.f)
    v = planck_f32(nu_at(j, pair_of(w.nu0), pair_of(w.dnu)), pair_of(w.theta), w.c1);
  w.out[j] = v;
}

// ------------------------------------------------------------ line sum tile
// Eq. (2) with the Eq. (1) strength ratio for one block: nu points from j0 on
// x kKappaCells cells starting at cell0.  Lines whose window meets the block's
// points are staged kLineTile at a time as line records (m, phi, the window's
// offsets -K + [phi > 0] and K, and per cell the Lorentz amplitude A = u S s
// gamma / (pi dnu^2) and the squared half width g2 = (gamma/dnu)^2), so that a
// line adds
//   A / ((j - r_i)^2 + g2)
// to kappa at point j.  Grid units: line i sits at r_i = (nu_i - nu0)/dnu =
// m_i + phi_i with integer m_i; the offset j - r_i is the exact float
// difference (j - m_i) minus phi_i, so no absolute-wavenumber cancellation
// occurs in FP32.  Window membership is the integer range
// [m_i - K + [phi_i > 0], m_i + K], the exact form of |j - r_i| <= K.
// Output: out[(cell - 0) * ld_out + (j - col0)] for col0 <= j < col_end;
// points at or beyond n_nu are written as 0.  Must be called by all threads of
// the block; `lds` holds kLineTile * kLineRec floats.
struct KappaTile {
  LineSet L;
  CellSet C;          // per-cell factors of this grid (row 0 = its first cell)
  int64_t n_cells;
  int n_nu;
  int K;
  int have_E;
  float* out;
  int64_t ld_out;
  int64_t col0;
  int64_t col_end;
  const int32_t* cell_list = nullptr;  // logical cell i -> cell_list[i] when set
  int compact_rows = 0;                // with a list: write row i instead of cell_list[i]
  int accumulate = 0;                  // add to the row instead of storing (a further gas)
  // the block sums part line_part of line_parts equal shares of the lines
  // its points need (its output is then a partial sum of the row)
  int line_parts = 1;
  int line_part = 0;
};

// Optional device-side gating of a launch of line-sum tiles, decided per
// block before any barrier: a block runs if its group of cells is marked
// with the current epoch in group_flag, or if one of the width-chunk_w
// spectral chunks its tile touches has chunk_err above tol.
struct TileGate {
  const unsigned* group_flag = nullptr;
  unsigned epoch = 0;
  const float* chunk_err = nullptr;
  float tol = 0;
  int chunk_w = 0;
  int n_chunks = 0;
};

// ------------------------------------------- line sum tile with far nodes
// The plain form's line sum.  Over a span of the grid a line whose window
// covers the span and whose centre lies far enough from the span's middle is
// smooth: it is evaluated at kFarNodes Chebyshev nodes of the span instead of
// at its points, and the nodes' sum over all such lines is interpolated once.
// Two levels: pairs of spans (128 points, centres at least 170.5 points from
// the middle) and spans (64 points, 84.5 points).  A pair's nodes are
// interpolated to the nodes of its two spans, theirs to the points.  With 12
// nodes of half width 31.6 (63.7) the interpolant of any A / (d^2 + g^2) is
// within 1.1e-7 of its value at the reach (poles at distance g from the real
// axis only help) and falls by a factor 10 per 12 points beyond it: below the
// reciprocal's rounding that every direct term carries.  Lines nearer, and
// those whose window ends inside the span, are summed point by point.
//
// Instructions per line and span of 8 cells: 28 point by point, 7 at a span's
// nodes, 3.5 at a pair's.  In a window of 1,001 points (cutoff 5 cm^-1 at
// 0.01) 16% of the lines that meet a span are near, 12% end inside it, 22%
// are at its nodes and 50% at the pair's.
//
// Issue-bound, as the sum at every point was, on 0.96 of the SIMD cycles.
// 24^3 cells, 20,000 points, 5,000 lines: 7.86 -> 3.38 ms, error against 64
// bits 3.1e-7 -> 1.5e-7 (fewer, shorter FP32 sums); 8^3 cells, 10,000 points,
// 20,000 lines: 1.85 -> 0.76 ms, 2.7e-6 -> 5.4e-7.  With the spans' level
// alone 3.80 and 0.94 ms.
constexpr int kFarNodes = 12;

struct FarTables {
  float node[2][kFarNodes];                       // offsets from the middle: span, pair
  alignas(16) float weight[64][kFarNodes];        // span's nodes -> its points
  alignas(16) float down[2][kFarNodes][kFarNodes];  // pair's nodes -> each span's nodes
};
constexpr FarTables make_far_tables() {
  // cos((2 k + 1) pi / 24)
  constexpr double c[6] = {0.99144486137381041, 0.92387953251128674, 0.79335334029123517,
                           0.60876142900872064, 0.38268343236508978, 0.13052619222005159};
  FarTables t{};
  double x[2][kFarNodes] = {};
  for (int v = 0; v < 2; ++v)
    for (int k = 0; k < 6; ++k) {
      x[v][k] = -(v ? 63.7 : 31.6) * c[k];
      x[v][kFarNodes - 1 - k] = (v ? 63.7 : 31.6) * c[k];
    }
  for (int v = 0; v < 2; ++v)
    for (int i = 0; i < kFarNodes; ++i) t.node[v][i] = (float)x[v][i];
  for (int i = 0; i < kFarNodes; ++i) {
    for (int j = 0; j < 64; ++j) {
      double w = 1.0;
      for (int k = 0; k < kFarNodes; ++k)
        if (k != i) w *= ((double)j - 31.5 - x[0][k]) / (x[0][i] - x[0][k]);
      t.weight[j][i] = (float)w;
    }
    for (int h = 0; h < 2; ++h)
      for (int j = 0; j < kFarNodes; ++j) {
        double w = 1.0;
        for (int k = 0; k < kFarNodes; ++k)
          if (k != i) w *= (x[0][j] + (h ? 32.0 : -32.0) - x[1][k]) / (x[1][i] - x[1][k]);
        t.down[h][j][i] = (float)w;
      }
  }
  return t;
}
static __device__ const FarTables far_tables = make_far_tables();
constexpr int kFarRef = kFarNodes / 2;  // the node the others are taken relative to
constexpr int kFarValues = kFarNodes * kKappaCells;
constexpr int kFarEntries = 2 * kFarValues + kKappaCells;  // LDS floats per wavefront

__device__ __forceinline__ void half_swap(float& a, float& b) {  // a's upper and b's lower half
  typedef unsigned U2 __attribute__((ext_vector_type(2)));
  const U2 r = __builtin_amdgcn_permlane32_swap((unsigned)__float_as_int(a),
                                                (unsigned)__float_as_int(b), false, false);
  a = __int_as_float((int)r.x);
  b = __int_as_float((int)r.y);
}
__device__ __forceinline__ void row_swap(float& a, float& b) {   // a's odd and b's even rows
  typedef unsigned U2 __attribute__((ext_vector_type(2)));
  const U2 r = __builtin_amdgcn_permlane16_swap((unsigned)__float_as_int(a),
                                                (unsigned)__float_as_int(b), false, false);
  a = __int_as_float((int)r.x);
  b = __int_as_float((int)r.y);
}

// Lane (s, c) = (lane >> 3, lane & 7) holds chain s of cell c for every node.
// Adds the eight chains, two nodes at a time, halving the registers at each
// step: lo gets node lane >> 3 of cell c, hi node 8 + (lane >> 3 & 3).
__device__ __forceinline__ void far_reduce(const float (&F)[kFarNodes], int lane, float& lo,
                                           float& hi) {
  float g[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const float a = F[2 * i] + dpp_f32<0x128>(F[2 * i]);  // row_ror:8
    const float b = F[2 * i + 1] + dpp_f32<0x128>(F[2 * i + 1]);
    g[i] = (lane & 8) ? b : a;
  }
  float s[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    row_swap(g[2 * i], g[2 * i + 1]);
    s[i] = g[2 * i] + g[2 * i + 1];
  }
  half_swap(s[0], s[1]);
  lo = s[0] + s[1];
  float t = s[2];
  half_swap(s[2], t);
  hi = s[2] + t;
}

// The node sums of a span (far_reduce's lo and hi) at its points, added to acc:
// points pt and pt + 32 for 4 cells (see kappa_tile_far).  Where a line's
// amplitude is beyond float every node holds the infinity that each point's term
// would be: the points take it from the node they are relative to, and the
// differences, which would be NaN, are left out.
__device__ __forceinline__ void far_points(float lo, float hi, int lane, float* fx,
                                           float (&acc)[2][4]) {
  constexpr int C = kKappaCells;
  const int pt = lane & 31, cg = lane >> 5;
  // the nodes relative to one of them: the interpolation's rounding then
  // scales with their differences
  const float ref = __int_as_float(
      __builtin_amdgcn_ds_bpermute(4 * (8 * kFarRef + (lane & 7)), __float_as_int(lo)));
  __builtin_amdgcn_wave_barrier();
  const float dlo = lo - ref, dhi = hi - ref;
  fx[lane] = __builtin_isfinite(dlo) ? dlo : 0.f;
  if (lane < 32) fx[64 + lane] = __builtin_isfinite(dhi) ? dhi : 0.f;
  if (lane < C) fx[2 * kFarValues + lane] = ref;
  __builtin_amdgcn_wave_barrier();
  float v[2][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) v[0][c] = v[1][c] = 0.f;
#pragma unroll
  for (int g = 0; g < kFarNodes / 4; ++g) {
    const float4 wl = *reinterpret_cast<const float4*>(&far_tables.weight[pt][4 * g]);
    const float4 wu = *reinterpret_cast<const float4*>(&far_tables.weight[pt + 32][4 * g]);
    const float l4[4] = {wl.x, wl.y, wl.z, wl.w}, u4[4] = {wu.x, wu.y, wu.z, wu.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float4 f = *reinterpret_cast<const float4*>(fx + (4 * g + k) * C + 4 * cg);
      const float f4[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        v[0][c] = fmaf(l4[k], f4[c], v[0][c]);
        v[1][c] = fmaf(u4[k], f4[c], v[1][c]);
      }
    }
  }
  const float4 rf = *reinterpret_cast<const float4*>(fx + 2 * kFarValues + 4 * cg);
  const float r4[4] = {rf.x, rf.y, rf.z, rf.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    acc[0][c] += r4[c] + v[0][c];
    acc[1][c] += r4[c] + v[1][c];
  }
}

// What a half of a span takes of a line: nothing, every point, the points
// from the window's first, up to its last, or within it.
constexpr int kNone = 0, kAll = 1, kFrom = 2, kUpTo = 3, kWithin = 4;
template <int M>
using Take = std::integral_constant<int, M>;

// Adds what point j takes of a line (header h) for 4 cells (parameters g0, g1).
template <int M>
__device__ __forceinline__ void add_half(const float4& h, const float4& g0, const float4& g1, float j,
                                         float (&s)[4]) {
  if constexpr (M == kNone) return;
  const float t = j - h.x;
  float d = t - h.y;
  if (M == kFrom) d = t >= h.z ? d : __builtin_inff();
  if (M == kUpTo) d = t <= h.w ? d : __builtin_inff();
  if (M == kWithin) d = ((t >= h.z) & (t <= h.w)) ? d : __builtin_inff();
  s[0] = fmaf(g0.x, fast_rcp(fmaf(d, d, g0.y)), s[0]);
  s[1] = fmaf(g0.z, fast_rcp(fmaf(d, d, g0.w)), s[1]);
  s[2] = fmaf(g1.x, fast_rcp(fmaf(d, d, g1.y)), s[2]);
  s[3] = fmaf(g1.z, fast_rcp(fmaf(d, d, g1.w)), s[3]);
}

// The plain form: points [j0, j0 + 256 SP) x kKappaCells
// cells; each wavefront owns SP spans of 64 points.  Point by point a lane
// takes points pt and pt + 32 of a span for 4 of the cells (2 LDS reads of
// parameters per line, where one point of 8 cells would take 4 and leave the
// LDS the bound); at the nodes it takes every eighth line for one cell.  A
// point's sum runs over the same lines in the same order, and a node's over
// the same lines in the same eight chains (by line index modulo 8), whatever
// SP and the staging are, so the values do not depend on them.
// lds: kLineTile * kLineRec floats; fx: this wavefront's kFarEntries floats.
// active (uniform over the wavefront): false leaves this wavefront's points
// untouched; it still stages line records with the others.
template <int SP>
__device__ void kappa_tile_far(const KappaTile& a, int j0, int64_t cell0, float* lds, float* fx,
                               bool active = true) {
  constexpr int C = kKappaCells;
  static_assert(kLineRec == 4 + 2 * C && 64 == 8 * C, "headers, then parameters of 8 cells");
  static_assert(SP == 1 || SP % 2 == 0, "a wavefront's spans are one of a pair, or whole pairs");
  constexpr FarTables tab = make_far_tables();
  constexpr int NP = (SP + 1) / 2;  // pairs a wavefront's spans lie in
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int pt = lane & 31, cg = lane >> 5;
  const int nl = a.L.n;
  auto bound = [&](const int4* table, int b, int k) {  // a scalar load: b is uniform
    return b < a.L.n_spans ? reinterpret_cast<const __attribute__((address_space(4))) int*>(
                                 reinterpret_cast<uintptr_t>(table))[4 * b + k]
                           : nl;
  };
  int blk_first = bound(a.L.span4, j0 / 64, 0);
  int blk_end = bound(a.L.span4, (j0 + kKappaThreads * SP - 1) / 64, 1);
  if (a.line_parts > 1) {
    const int share = (blk_end - blk_first + a.line_parts - 1) / a.line_parts;
    blk_first = min(blk_end, blk_first + a.line_part * share);
    blk_end = min(blk_end, blk_first + share);
  }
  // cuts of the sorted list.  Per pair: the lines at its nodes, [p0, p1) below
  // and [p2, p3) above.  Per span: lines ending inside it [x, c0), of which
  // [x, h0) meet its lower half only and [x, s0) also start at or before it
  // (all, but for windows narrower than the span); covering ones [c0, c1), of
  // which [m0, m1) are near; starting inside it [c1, y), of which [h1, y) meet
  // its upper half only
  struct Pair4 {
    int p0, p1, p2, p3;
  } pair[NP];
  struct Cuts {
    int x, h0, s0, c0, m0, m1, c1, h1, y;
  } cut[SP];
  const int wj0 = j0 + wave * 64 * SP;
#pragma unroll
  for (int v = 0; v < NP; ++v) {
    const int b = (wj0 / 128 + v) * 2;
    Pair4 q;
    q.p1 = bound(a.L.span_pair, b / 2, 0);
    q.p0 = min(bound(a.L.span4, b + 1, 2), q.p1);
    q.p2 = bound(a.L.span_pair, b / 2, 1);
    q.p3 = max(bound(a.L.span4, b, 3), q.p2);
    pair[v] = q;
  }
#pragma unroll
  for (int p = 0; p < SP; ++p) {
    const int b = wj0 / 64 + p;
    Cuts q;
    q.x = bound(a.L.span4, b, 0);
    q.y = bound(a.L.span4, b, 1);
    q.c0 = min(max(bound(a.L.span4, b, 2), q.x), q.y);
    q.c1 = max(q.c0, min(bound(a.L.span4, b, 3), q.y));
    q.m0 = min(max(bound(a.L.span_far, b, 0), q.c0), q.c1);
    q.m1 = min(max(bound(a.L.span_far, b, 1), q.m0), q.c1);
    q.s0 = min(max(bound(a.L.span4, b, 3), q.x), q.c0);
    q.h0 = min(max(bound(a.L.span_far, b, 2), q.x), q.s0);
    q.h1 = min(max(bound(a.L.span_far, b, 3), q.c1), q.y);
    cut[p] = q;
  }

  float acc[SP][2][4];
  float F[SP][kFarNodes], F2[NP][kFarNodes];
#pragma unroll
  for (int p = 0; p < SP; ++p) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[p][h][c] = 0.f;
#pragma unroll
    for (int n = 0; n < kFarNodes; ++n) F[p][n] = 0.f;
  }
#pragma unroll
  for (int v = 0; v < NP; ++v)
#pragma unroll
    for (int n = 0; n < kFarNodes; ++n) F2[v][n] = 0.f;

  // staging: a thread forms the parameters of every 32nd line for one cell,
  // whose factors it keeps; headers (m, phi, lo, hi) and parameters lie apart,
  // so that eight lines' parameters of eight cells are 512 contiguous bytes
  float4* hdr = reinterpret_cast<float4*>(lds);
  float2* par = reinterpret_cast<float2*>(lds + 4 * kLineTile);
  const int cc = tid % C;
  CellFactors cf;
  {
    int64_t scell = cell0 + cc;
    if (scell >= a.n_cells) scell = a.n_cells - 1;
    if (a.cell_list) scell = a.cell_list[scell];
    cf = CellFactors{a.C.beta[scell], a.C.theta[scell], a.C.G[scell], a.C.P[scell],
                     a.C.lam2[scell]};
  }

  for (int base = blk_first & ~7; base < blk_end; base += kLineTile) {
    const int nt = min(kLineTile, blk_end - base);
    __syncthreads();
#pragma unroll 2
    for (int li = tid / C; li < nt; li += kKappaThreads / C) {
      const LineData d = a.L.data[base + li];
      if (cc == 0) hdr[li] = make_float4(d.m, d.phi, d.lo, (float)a.K);
      float amp, g2;
      line_cell_params(d, cf, a.have_E, amp, g2);
      par[li * C + cc] = make_float2(amp, g2);
    }
    __syncthreads();
    if (!active) continue;
    const int first = max(base, blk_first), end = base + nt;
    // lines [l0, l1) at the nodes `node` about the point v0 + mid
    auto far = [&](float (&f)[kFarNodes], const float (&node)[kFarNodes], float v0, float mid,
                   int l0, int l1) {
      l0 = __builtin_amdgcn_readfirstlane(max(l0, first) - base);
      l1 = __builtin_amdgcn_readfirstlane(min(l1, end) - base);
      for (int l8 = l0 & ~7; l8 < l1; l8 += 8) {  // base: a multiple of 8
        const int l = l8 + (lane >> 3);
        if (l >= l0 && l < l1) {
          const float2 h = *reinterpret_cast<const float2*>(hdr + l);
          const float2 ag = par[l8 * C + lane];
          const float e = ((h.x - v0) - mid) + h.y;  // the centre from the middle
#pragma unroll
          for (int n = 0; n < kFarNodes; ++n) {
            const float d = node[n] - e;
            f[n] = fmaf(ag.x, fast_rcp(fmaf(d, d, ag.y)), f[n]);
          }
        }
      }
    };
#pragma unroll
    for (int v = 0; v < NP; ++v) {
      const float v0 = (float)((wj0 / 128 + v) * 128);
      far(F2[v], tab.node[1], v0, 63.5f, pair[v].p0, pair[v].p1);
      far(F2[v], tab.node[1], v0, 63.5f, pair[v].p2, pair[v].p3);
    }
#pragma unroll
    for (int p = 0; p < SP; ++p) {
      const float v0 = (float)(wj0 + 64 * p);
      const float jl = v0 + (float)pt, ju = jl + 32.f;
      // lines [l0, l1) point by point: what the lower and the upper half take
      // of them
      auto direct = [&](auto lower, auto upper, int l0, int l1) {
        l0 = __builtin_amdgcn_readfirstlane(max(l0, first) - base);
        l1 = __builtin_amdgcn_readfirstlane(min(l1, end) - base);
        for (int l = l0; l < l1; ++l) {
          const float4 h = hdr[l];
          const float4* g = reinterpret_cast<const float4*>(par + l * C + 4 * cg);
          const float4 g0 = g[0], g1 = g[1];
          add_half<decltype(lower)::value>(h, g0, g1, jl, acc[p][0]);
          add_half<decltype(upper)::value>(h, g0, g1, ju, acc[p][1]);
        }
      };
      const Cuts& q = cut[p];
      const Pair4& r = pair[p / 2];
      direct(Take<kUpTo>(), Take<kNone>(), q.x, q.h0);
      direct(Take<kAll>(), Take<kUpTo>(), q.h0, q.s0);
      direct(Take<kWithin>(), Take<kWithin>(), q.s0, q.c0);
      far(F[p], tab.node[0], v0, 31.5f, q.c0, min(r.p0, q.m0));
      far(F[p], tab.node[0], v0, 31.5f, max(r.p1, q.c0), q.m0);
      direct(Take<kAll>(), Take<kAll>(), q.m0, q.m1);
      far(F[p], tab.node[0], v0, 31.5f, q.m1, min(r.p2, q.c1));
      far(F[p], tab.node[0], v0, 31.5f, max(r.p3, q.m1), q.c1);
      direct(Take<kFrom>(), Take<kAll>(), q.c1, q.h1);
      direct(Take<kNone>(), Take<kFrom>(), q.h1, q.y);
    }
  }
  if (!active) return;

  const int n_hi = 8 + ((lane >> 3) & 3);  // the node of far_reduce's hi
#pragma unroll
  for (int p = 0; p < SP; ++p) {
    const Pair4& r = pair[p / 2];
    const bool paired = r.p1 - r.p0 + r.p3 - r.p2 > 0;
    if (!paired && cut[p].m0 - cut[p].c0 + cut[p].c1 - cut[p].m1 == 0) continue;  // no far line
    if (paired && p % 2 == 0) {  // the pair's node sums, for both of its spans
      float lo, hi;
      far_reduce(F2[p / 2], lane, lo, hi);
      __builtin_amdgcn_wave_barrier();
      fx[kFarValues + lane] = lo;
      if (lane < 32) fx[kFarValues + 64 + lane] = hi;
      __builtin_amdgcn_wave_barrier();
    }
    float lo, hi;
    far_reduce(F[p], lane, lo, hi);
    if (paired) {
      const int half = (wj0 / 64 + p) & 1;
      const float* dl = far_tables.down[half][lane >> 3];
      const float* dh = far_tables.down[half][n_hi];
      const float lo0 = lo, hi0 = hi;
#pragma unroll
      for (int k = 0; k < kFarNodes; ++k) {
        const float f = fx[kFarValues + k * C + (lane & 7)];
        lo = fmaf(dl[k], f, lo);
        hi = fmaf(dh[k], f, hi);
      }
      // an infinity at the pair's nodes (see far_points)
      const float f = fx[kFarValues + kFarRef * C + (lane & 7)];
      if (!__builtin_isfinite(lo)) lo = lo0 + f;
      if (!__builtin_isfinite(hi)) hi = hi0 + f;
    }
    far_points(lo, hi, lane, fx, acc[p]);
  }

#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int64_t cell = cell0 + 4 * cg + c;
    if (cell >= a.n_cells) break;
    if (a.cell_list && !a.compact_rows) cell = a.cell_list[cell];
#pragma unroll
    for (int p = 0; p < SP; ++p)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t j = wj0 + 64 * p + 32 * h + pt;
        if (j >= a.col0 && j < a.col_end) {
          float* o = a.out + cell * a.ld_out + (j - a.col0);
          const float v = acc[p][h][c];
          *o = (j < a.n_nu) ? (a.accumulate ? *o + v : v) : 0.f;
        }
      }
  }
}

// ------------------------------------------------- the precision form's line sum
// Points [j0, j0 + 512) x kKappaCells cells, every line at every point, with line
// records from line_cell_params_f32; 512 threads, a span of 64 points per
// wavefront, each lane points pt and pt + 32 for 4 cells.
//
// The order of additions is fixed: the lines of a run of 128 points are taken a
// stage of 256 at a time, in three ranges (windows that end in the run, cover it,
// start in it), each range in blocks of 16 lines that are summed plainly and
// folded in with TwoSum.  A span belongs to a run of 128 points and follows its
// blocks, and takes of a block the lines that meet it: the others would add zeros.
//
// Issue-bound (0.96 of the issue slots).  One span a wavefront instead of two
// passes over the lines that miss it and leaves room for six wavefronts per
// SIMD (three blocks, each two on every SIMD) instead of five, and eight wavefronts
// share a stage as four of two spans did.  A call with its Planck table, two spans -> one: 16^3 cells, 20,000 points,
// 5,000 lines 2.81 -> 2.73 ms; 12^3 cells, 12,000 points, 78,000 lines in windows
// of 200 points 9.67 -> 6.17 ms, 3,000 lines in windows of 1000 points 0.82 ->
// 0.77 ms; 5 x 6 x 7 cells, 3,037 points, 760 lines 0.096 -> 0.070 ms.  16^3 cells
// and 14,000 points with windows of 2000, which few lines miss, 1.83 -> 1.85 ms.
constexpr int kPrecThreads = 512;
__device__ inline void kappa_tile(const KappaTile& a, int j0, int64_t cell0, float* lds) {
  constexpr int C = kKappaCells;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int pt = lane & 31, cg = lane >> 5;
  const int nl = a.L.n;
  auto bound = [&](const int4* table, int b, int k) {  // a scalar load: b is uniform
    return b < a.L.n_spans ? reinterpret_cast<const __attribute__((address_space(4))) int*>(
                                 reinterpret_cast<uintptr_t>(table))[4 * b + k]
                           : nl;
  };
  const int blk_first = bound(a.L.span4, j0 / 64, 0);
  const int blk_end = bound(a.L.span4, (j0 + 511) / 64, 1);
  // the run of 128 points: its lines, and those covering it
  const int wj0 = j0 + wave * 64, b = wj0 / 64, r = (j0 + (wave >> 1) * 128) / 64;
  const int w_first = bound(a.L.span4, r, 0), w_end = bound(a.L.span4, r + 1, 1);
  const int f_first = bound(a.L.span4, r + 1, 2), f_end = bound(a.L.span4, r, 3);
  // the span's cuts (see kappa_tile_far)
  const int x = bound(a.L.span4, b, 0), y = bound(a.L.span4, b, 1);
  const int c0 = min(max(bound(a.L.span4, b, 2), x), y);
  const int c1 = max(c0, min(bound(a.L.span4, b, 3), y));
  const int s0 = min(max(bound(a.L.span4, b, 3), x), c0);
  const int h0 = min(max(bound(a.L.span_far, b, 2), x), s0);
  const int h1 = min(max(bound(a.L.span_far, b, 3), c1), y);

  float acc[2][4], cmp[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[h][c] = cmp[h][c] = 0.f;
  float4* hdr = reinterpret_cast<float4*>(lds);
  float2* par = reinterpret_cast<float2*>(lds + 4 * kLineTile);
  const int cc = tid % C;
  CellFactors32 cf;
  {
    int64_t scell = cell0 + cc;
    if (scell >= a.n_cells) scell = a.n_cells - 1;
    if (a.cell_list) scell = a.cell_list[scell];
    cf = CellFactors32{a.C.beta2[scell], a.C.theta2[scell], a.C.Gq[scell], a.C.Pf[scell],
                       a.C.lamf[scell]};
  }
  const float jl = (float)wj0 + (float)pt, ju = jl + 32.f;

  for (int base = blk_first; base < blk_end; base += kLineTile) {
    const int nt = min(kLineTile, blk_end - base);
    __syncthreads();
    for (int li = tid / C; li < nt; li += kPrecThreads / C) {
      const int i = base + li;
      if (cc == 0) {
        const int m = a.L.m[i];
        hdr[li] = make_float4((float)m, a.L.phi[i], (float)(a.L.wlo[i] - m), (float)a.K);
      }
      float amp, g2;
      line_cell_params_f32(a.L, cf, i, a.have_E, amp, g2);
      par[li * C + cc] = make_float2(amp, g2);
    }
    __syncthreads();
    const int lb = max(base, w_first), le = min(base + nt, w_end);
    const int fb = min(le, max(lb, f_first)), fe = max(fb, min(le, f_end));
    auto range = [&](int r0, int r1) {
      const int first = max(r0, x), end = min(r1, y);
      for (int g = r0 + ((first - r0) & ~15); g < end; g += 16) {  // the blocks that meet the span
        const int g0 = max(g, first), g1 = min(g + 16, end);
        float part[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) part[h][c] = 0.f;
        auto direct = [&](auto lower, auto upper, int l0, int l1) {
          l0 = __builtin_amdgcn_readfirstlane(max(l0, g0) - base);
          l1 = __builtin_amdgcn_readfirstlane(min(l1, g1) - base);
          for (int l = l0; l < l1; ++l) {
            const float4 h = hdr[l];
            const float4* g = reinterpret_cast<const float4*>(par + l * C + 4 * cg);
            const float4 p0 = g[0], p1 = g[1];
            add_half<decltype(lower)::value>(h, p0, p1, jl, part[0]);
            add_half<decltype(upper)::value>(h, p0, p1, ju, part[1]);
          }
        };
        if (g0 >= c0 && g1 <= c1) {
          direct(Take<kAll>(), Take<kAll>(), c0, c1);
        } else {
          direct(Take<kUpTo>(), Take<kNone>(), x, h0);
          direct(Take<kAll>(), Take<kUpTo>(), h0, s0);
          direct(Take<kWithin>(), Take<kWithin>(), s0, c0);
          direct(Take<kAll>(), Take<kAll>(), c0, c1);
          direct(Take<kFrom>(), Take<kAll>(), c1, h1);
          direct(Take<kNone>(), Take<kFrom>(), h1, y);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) two_sum_acc(acc[h][c], cmp[h][c], part[h][c]);
      }
    };
    range(lb, fb);
    range(fb, fe);
    range(fe, le);
  }

#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int64_t cell = cell0 + 4 * cg + c;
    if (cell >= a.n_cells) break;
    if (a.cell_list && !a.compact_rows) cell = a.cell_list[cell];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t j = wj0 + 32 * h + pt;
      if (j >= a.col0 && j < a.col_end) {
        const float v = acc[h][c] + cmp[h][c];
        float* o = a.out + cell * a.ld_out + (j - a.col0);
        *o = (j < a.n_nu) ? (a.accumulate ? *o + v : v) : 0.f;
      }
    }
  }
}

// -------------------------------------------- the compensated sum with far nodes
// Lane (s, c) holds chain s of cell c for every node; adds the eight chains in
// FP64, as far_reduce.
__device__ __forceinline__ void row_swap64(double& a, double& b) {
  float2 x = *reinterpret_cast<float2*>(&a), y = *reinterpret_cast<float2*>(&b);
  row_swap(x.x, y.x);
  row_swap(x.y, y.y);
  a = *reinterpret_cast<double*>(&x);
  b = *reinterpret_cast<double*>(&y);
}
__device__ __forceinline__ void half_swap64(double& a, double& b) {
  float2 x = *reinterpret_cast<float2*>(&a), y = *reinterpret_cast<float2*>(&b);
  half_swap(x.x, y.x);
  half_swap(x.y, y.y);
  a = *reinterpret_cast<double*>(&x);
  b = *reinterpret_cast<double*>(&y);
}
__device__ __forceinline__ void far_reduce64(const float (&F)[kFarNodes], const float (&E)[kFarNodes],
                                             int lane, double& lo, double& hi) {
  double g[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    double a = (double)F[2 * i] + (double)E[2 * i];
    double b = (double)F[2 * i + 1] + (double)E[2 * i + 1];
    a += dpp_f64<0x128>(a);  // row_ror:8
    b += dpp_f64<0x128>(b);
    g[i] = (lane & 8) ? b : a;
  }
  double s[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    row_swap64(g[2 * i], g[2 * i + 1]);
    s[i] = g[2 * i] + g[2 * i + 1];
  }
  half_swap64(s[0], s[1]);
  lo = s[0] + s[1];
  double t = s[2];
  half_swap64(s[2], t);
  hi = s[2] + t;
}

struct FarWeights64 {
  alignas(16) double weight[64][kFarNodes];  // FarTables::weight for these nodes
};
constexpr FarWeights64 make_far_weights64() {
  constexpr FarTables f = make_far_tables();
  FarWeights64 t{};
  for (int i = 0; i < kFarNodes; ++i)
    for (int j = 0; j < 64; ++j) {
      double w = 1.0;
      for (int k = 0; k < kFarNodes; ++k)
        if (k != i)
          w *= ((double)j - 31.5 - (double)f.node[0][k]) / ((double)f.node[0][i] - (double)f.node[0][k]);
      t.weight[j][i] = w;
    }
  return t;
}
static __device__ const FarWeights64 far_weights64 = make_far_weights64();
constexpr int kCompEntries = kFarValues;  // LDS doubles per wavefront

// The compensated sum of the batched launches, with the plain form's line
// parameters: points [j0, j0 + 256) x kKappaCells cells, a span of 64 points per
// wavefront.  Runs of up to 8 lines point by point (32 at the nodes, in eight
// chains) are summed plainly and folded in with TwoSum; the chains are added and
// the nodes interpolated in FP64, so the result is rounded once.  The span's
// nodes alone are used (a wavefront with one span would not share a pair's).
// lds: kLineTile * kLineRec floats; fx: this wavefront's kCompEntries doubles.
// (The precision form keeps kappa_tile: its powers are FP64 sums, and another
// order of additions, which changes a table's last bit at one point in five,
// would move them by up to 2e-9 at 1,500 points.)
//
// Issue-bound.  16^3 cells, 20,000 points, 5,000 lines: 2.75 -> 1.42 ms.  Error
// against 64 bits (rms over the points, 3 to 200 lines per cm^-1, steps of 0.005
// to 0.05): 7.2e-8 to 9.5e-8, every line at every point 7.8e-8 to 1.1e-7.
__device__ inline void kappa_tile_comp(const KappaTile& a, int j0, int64_t cell0, float* lds, double* fx) {
  constexpr int C = kKappaCells;
  constexpr FarTables tab = make_far_tables();
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int pt = lane & 31, cg = lane >> 5;
  const int nl = a.L.n;
  auto bound = [&](const int4* table, int b, int k) {  // a scalar load: b is uniform
    return b < a.L.n_spans ? reinterpret_cast<const __attribute__((address_space(4))) int*>(
                                 reinterpret_cast<uintptr_t>(table))[4 * b + k]
                           : nl;
  };
  const int blk_first = bound(a.L.span4, j0 / 64, 0);
  const int blk_end = bound(a.L.span4, (j0 + kKappaThreads - 1) / 64, 1);
  // the span's cuts, as kappa_tile_far's
  const int wj0 = j0 + wave * 64, b = wj0 / 64;
  const int x = bound(a.L.span4, b, 0), y = bound(a.L.span4, b, 1);
  const int c0 = min(max(bound(a.L.span4, b, 2), x), y);
  const int c1 = max(c0, min(bound(a.L.span4, b, 3), y));
  const int m0 = min(max(bound(a.L.span_far, b, 0), c0), c1);
  const int m1 = min(max(bound(a.L.span_far, b, 1), m0), c1);
  const int s0 = min(max(bound(a.L.span4, b, 3), x), c0);
  const int h0 = min(max(bound(a.L.span_far, b, 2), x), s0);
  const int h1 = min(max(bound(a.L.span_far, b, 3), c1), y);

  float acc[2][4], cmp[2][4], F[kFarNodes], E[kFarNodes];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[h][c] = cmp[h][c] = 0.f;
#pragma unroll
  for (int n = 0; n < kFarNodes; ++n) F[n] = E[n] = 0.f;

  float4* hdr = reinterpret_cast<float4*>(lds);
  float2* par = reinterpret_cast<float2*>(lds + 4 * kLineTile);
  const int cc = tid % C;
  CellFactors cf;
  {
    int64_t scell = cell0 + cc;
    if (scell >= a.n_cells) scell = a.n_cells - 1;
    if (a.cell_list) scell = a.cell_list[scell];
    cf = CellFactors{a.C.beta[scell], a.C.theta[scell], a.C.G[scell], a.C.P[scell],
                     a.C.lam2[scell]};
  }
  const float v0 = (float)wj0;
  const float jl = v0 + (float)pt, ju = jl + 32.f;

  for (int base = blk_first & ~7; base < blk_end; base += kLineTile) {
    const int nt = min(kLineTile, blk_end - base);
    __syncthreads();
#pragma unroll 2
    for (int li = tid / C; li < nt; li += kKappaThreads / C) {
      const LineData d = a.L.data[base + li];
      if (cc == 0) hdr[li] = make_float4(d.m, d.phi, d.lo, (float)a.K);
      float amp, g2;
      line_cell_params(d, cf, a.have_E, amp, g2);
      par[li * C + cc] = make_float2(amp, g2);
    }
    __syncthreads();
    const int first = max(base, blk_first), end = base + nt;
    auto direct = [&](auto lower, auto upper, int l0, int l1) {
      l0 = __builtin_amdgcn_readfirstlane(max(l0, first) - base);
      l1 = __builtin_amdgcn_readfirstlane(min(l1, end) - base);
      while (l0 < l1) {
        const int le = min(l0 + 8, l1);
        float part[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) part[h][c] = 0.f;
        for (int l = l0; l < le; ++l) {
          const float4 h = hdr[l];
          const float4* g = reinterpret_cast<const float4*>(par + l * C + 4 * cg);
          const float4 g0 = g[0], g1 = g[1];
          add_half<decltype(lower)::value>(h, g0, g1, jl, part[0]);
          add_half<decltype(upper)::value>(h, g0, g1, ju, part[1]);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (decltype(lower)::value != kNone) two_sum_acc(acc[0][c], cmp[0][c], part[0][c]);
          if (decltype(upper)::value != kNone) two_sum_acc(acc[1][c], cmp[1][c], part[1][c]);
        }
        l0 = le;
      }
    };
    direct(Take<kUpTo>(), Take<kNone>(), x, h0);
    direct(Take<kAll>(), Take<kUpTo>(), h0, s0);
    direct(Take<kWithin>(), Take<kWithin>(), s0, c0);
    direct(Take<kAll>(), Take<kAll>(), m0, m1);
    direct(Take<kFrom>(), Take<kAll>(), c1, h1);
    direct(Take<kNone>(), Take<kFrom>(), h1, y);
    if (c0 < m0 || m1 < c1) {
      float part[kFarNodes];
#pragma unroll
      for (int n = 0; n < kFarNodes; ++n) part[n] = 0.f;
      auto far = [&](int l0, int l1) {
        l0 = __builtin_amdgcn_readfirstlane(max(l0, first) - base);
        l1 = __builtin_amdgcn_readfirstlane(min(l1, end) - base);
        for (int l8 = l0 & ~7; l8 < l1; l8 += 8) {  // base: a multiple of 8
          const int l = l8 + (lane >> 3);
          if (l >= l0 && l < l1) {
            const float2 h = *reinterpret_cast<const float2*>(hdr + l);
            const float2 ag = par[l8 * C + lane];
            const float e = ((h.x - v0) - 31.5f) + h.y;  // the centre from the middle
#pragma unroll
            for (int n = 0; n < kFarNodes; ++n) {
              const float d = tab.node[0][n] - e;
              part[n] = fmaf(ag.x, fast_rcp(fmaf(d, d, ag.y)), part[n]);
            }
          }
        }
      };
      far(c0, m0);
      far(m1, c1);
#pragma unroll
      for (int n = 0; n < kFarNodes; ++n) two_sum_acc(F[n], E[n], part[n]);
    }
  }

  double v[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < 4; ++c) v[h][c] = (double)acc[h][c] + (double)cmp[h][c];
  if (c0 < m0 || m1 < c1) {
    double lo, hi;
    far_reduce64(F, E, lane, lo, hi);
    __builtin_amdgcn_wave_barrier();
    fx[lane] = lo;
    if (lane < 32) fx[64 + lane] = hi;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int n = 0; n < kFarNodes; n += 2) {
      const double2 wl = *reinterpret_cast<const double2*>(&far_weights64.weight[pt][n]);
      const double2 wu = *reinterpret_cast<const double2*>(&far_weights64.weight[pt + 32][n]);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double* f = fx + (n + k) * C + 4 * cg;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          v[0][c] = fma(k ? wl.y : wl.x, f[c], v[0][c]);
          v[1][c] = fma(k ? wu.y : wu.x, f[c], v[1][c]);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();  // a next call writes fx
  }

#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int64_t cell = cell0 + 4 * cg + c;
    if (cell >= a.n_cells) break;
    if (a.cell_list && !a.compact_rows) cell = a.cell_list[cell];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t j = wj0 + 32 * h + pt;
      if (j >= a.col0 && j < a.col_end) {
        float* o = a.out + cell * a.ld_out + (j - a.col0);
        const float r = (float)v[h][c];
        *o = (j < a.n_nu) ? (a.accumulate ? *o + r : r) : 0.f;
      }
    }
  }
}

// ------------------------------------------------------------ Philox4x64-10
// Salmon et al., SC'11: ten rounds of two 64x64->128 products by the round
// multipliers, high halves xored with the other words and the key, with a
// Weyl key bump between rounds.
__device__ __forceinline__ void philox4x64_10(uint64_t x[4], uint64_t k0, uint64_t k1) {
  const uint64_t m0 = 0xD2E7470EE14C6C93ULL, m1 = 0xCA5A826395121157ULL;
  const uint64_t w0 = 0x9E3779B97F4A7C15ULL, w1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t lo0 = m0 * x[0], hi0 = __umul64hi(m0, x[0]);
    const uint64_t lo1 = m1 * x[2], hi1 = __umul64hi(m1, x[2]);
    const uint64_t y0 = hi1 ^ x[1] ^ k0;
    const uint64_t y2 = hi0 ^ x[3] ^ k1;
    x[0] = y0; x[1] = lo1; x[2] = y2; x[3] = lo0;
    k0 += w0; k1 += w1;
  }
}

__device__ __forceinline__ int64_t isqrt64(int64_t v) {  // floor(sqrt(v)), v < 2^50
  int64_t s = (int64_t)sqrt((double)v);
  while (s * s > v) --s;
  while ((s + 1) * (s + 1) <= v) ++s;
  return s;
}

// Ray r of the set drawn with `seed`: key (seed, 1), counter (r, block, 0, 0).
// Block 0: word 0 picks the face with probability proportional to its area,
// words 1-2 the odd in-face fixed-point coordinates, word 3 the first disk
// candidate; blocks 1..15 give further candidates, four per block.  A
// candidate word gives two 21-bit signed integers (A, B), accepted when
// A^2 + B^2 < 2^40; the inward component is isqrt(2^40 - A^2 - B^2).
__device__ inline void sample_ray(uint64_t seed, uint64_t r, int nx, int ny, int nz,
                                  int64_t O[3], int64_t D[3]) {
  const int64_t n[3] = {nx, ny, nz};
  uint64_t w[4] = {r, 0, 0, 0};
  philox4x64_10(w, seed, 1);
  const uint64_t ax = (uint64_t)(ny) * nz, ay = (uint64_t)(nz) * nx, az = (uint64_t)(nx) * ny;
  const uint64_t total = 2 * (ax + ay + az);
  const uint64_t u = __umul64hi(w[0], total);
  int face;
  if (u < ax) face = 0;
  else if (u < 2 * ax) face = 1;
  else if (u < 2 * ax + ay) face = 2;
  else if (u < 2 * ax + 2 * ay) face = 3;
  else if (u < 2 * ax + 2 * ay + az) face = 4;
  else face = 5;
  const int axis = face >> 1, side = face & 1;
  const int t1 = (axis + 1) % 3, t2 = (axis + 2) % 3;
  O[axis] = side ? n[axis] * kCellUnits : 0;
  O[t1] = 2 * (int64_t)__umul64hi(w[1], (uint64_t)n[t1] << 20) + 1;
  O[t2] = 2 * (int64_t)__umul64hi(w[2], (uint64_t)n[t2] << 20) + 1;

  const int64_t R = int64_t(1) << 20, R2 = R * R, M21 = (int64_t(1) << 21) - 1;
  int64_t A = 0, B = 0;
  uint64_t cand = w[3];
  for (int k = 0; k < 61; ++k) {
    if (k > 0) {
      const int pos = (k - 1) & 3;
      if (pos == 0) {
        w[0] = r; w[1] = (uint64_t)(1 + ((k - 1) >> 2)); w[2] = 0; w[3] = 0;
        philox4x64_10(w, seed, 1);
      }
      cand = w[pos];
    }
    const int64_t a = (int64_t)(cand & (uint64_t)M21) - R;
    const int64_t b = (int64_t)((cand >> 21) & (uint64_t)M21) - R;
    if (a * a + b * b < R2) { A = a; B = b; break; }
  }
  const int64_t Cn = isqrt64(R2 - A * A - B * B);
  D[axis] = side ? -Cn : Cn;
  D[t1] = A;
  D[t2] = B;
}

// Incremental traversal with exact integer comparisons.  The parameter of
// the next plane along axis k is tnum_k / tden_k (tden_k = |D_k| <= 2^21,
// tnum_k <= 2^41); the smallest one is found by cross-multiplication, every
// axis reaching it steps at once (edges and corners are crossed in one step),
// and the segment length is the exact integer numerator of t_next - t_prev
// over its denominator, times |D| h / 2^21, rounded once to FP32.  An axis the
// ray does not move along keeps 1 / 0, later than every plane.
//
// The chain of a step is what it costs, a wavefront having few others beside
// it: the three pairs are compared once, for the smallest and for the ties
// alike, in products of 64 by 32 bits.  Ray generation and traversal of 1024
// rays, 8^3 cells: 10.1 us, 4096 rays, 24^3 cells: 25.5, 2^20 rays, 32^3 cells:
// 259 (two passes over the axes with 64 by 64 products: 15.5, 42.8 and 319).
__device__ inline int traverse(int nx, int ny, int nz, double unit_cm, const int64_t O[3],
                               const int64_t D[3], int max_segs, int2* out) {
  const unsigned n[3] = {(unsigned)nx, (unsigned)ny, (unsigned)nz};
  unsigned idx[3], den[3];
  uint64_t num[3];
  for (int k = 0; k < 3; ++k) {
    const int64_t q = O[k] / kCellUnits;  // O >= 0
    const bool on_plane = (O[k] % kCellUnits) == 0;
    const int64_t i = (on_plane && D[k] < 0) ? q - 1 : q;
    idx[k] = (unsigned)i;  // -1: beyond every n
    den[k] = (unsigned)(D[k] < 0 ? -D[k] : D[k]);
    if (D[k] > 0) num[k] = (uint64_t)((i + 1) * kCellUnits - O[k]);
    else if (D[k] < 0) num[k] = (uint64_t)(O[k] - i * kCellUnits);
    else num[k] = 1;
  }
  const unsigned d0 = den[0], d1 = den[1], d2 = den[2];
  const unsigned step0 = D[0] > 0 ? 1u : ~0u, step1 = D[1] > 0 ? 1u : ~0u, step2 = D[2] > 0 ? 1u : ~0u;
  unsigned i0 = idx[0], i1 = idx[1], i2 = idx[2];
  uint64_t t0 = num[0], t1 = num[1], t2 = num[2];
  const double dlen = sqrt((double)D[0] * (double)D[0] + (double)D[1] * (double)D[1] +
                           (double)D[2] * (double)D[2]);
  uint64_t pnum = 0;
  unsigned pden = 1;
  int count = 0;
  while (i0 < n[0] && i1 < n[1] && i2 < n[2] && count < max_segs) {
    const uint64_t a01 = t0 * d1, b01 = t1 * d0, a02 = t0 * d2, b02 = t2 * d0, a12 = t1 * d2,
                   b12 = t2 * d1;
    // the first of the axes with the smallest parameter, and those it ties with
    const bool m0 = a01 <= b01 && a02 <= b02;
    const bool m1 = !m0 && a12 <= b12;
    const bool go1 = m0 ? a01 == b01 : m1;
    const bool go2 = m0 ? a02 == b02 : (m1 ? a12 == b12 : true);
    const uint64_t mnum = m0 ? t0 : (m1 ? t1 : t2);
    const unsigned mden = m0 ? d0 : (m1 ? d1 : d2);
    const int64_t dnum = (int64_t)(mnum * pden - pnum * mden);
    const int64_t dden = (int64_t)((uint64_t)mden * pden);
    const double len = ((double)dnum / (double)dden) * dlen * unit_cm;
    const int cell = (int)(i0 + n[0] * (i1 + n[1] * i2));
    out[count] = make_int2(cell, __float_as_int((float)len));
    ++count;
    i0 += m0 ? step0 : 0u;
    t0 += m0 ? (uint64_t)kCellUnits : 0;
    i1 += go1 ? step1 : 0u;
    t1 += go1 ? (uint64_t)kCellUnits : 0;
    i2 += go2 ? step2 : 0u;
    t2 += go2 ? (uint64_t)kCellUnits : 0;
    pnum = mnum;
    pden = mden;
  }
  return count;
}

// ------------------------------------------------------------ ray order
// Rays that run nearly parallel through nearby cells read the same kappa
// rows.  Marching them together (and on one XCD, see march_kernel) lets those
// rows be served from L2 instead of beyond it.  The key is the dominant axis
// and sign of D, a 3 x 3 bin of the two transverse direction ratios, and the
// Morton index (6 bits per axis) of the point where the ray's line crosses
// the grid's mid-plane normal to the dominant axis, over [-N, 2N] cells.
// The order changes only the order of the FP64 tally additions.
__device__ __forceinline__ uint32_t spread6(uint32_t v) {  // bits 0..5 -> even bits
  v = (v | (v << 4)) & 0x30fu;
  v = (v | (v << 2)) & 0x333u;
  v = (v | (v << 1)) & 0x555u;
  return v;
}

__device__ inline uint32_t order_key(const int64_t O[3], const int64_t D[3], int nx, int ny, int nz) {
  const int64_t n[3] = {nx, ny, nz};
  int ax = 0;
  for (int k = 1; k < 3; ++k)
    if (llabs(D[k]) > llabs(D[ax])) ax = k;
  const int a1 = ax == 2 ? 0 : ax + 1, a2 = ax == 0 ? 2 : ax - 1;
  const double dax = (double)D[ax];
  const double inv = 1.0 / fabs(dax);
  const int b1 = min(2, (int)(((double)D[a1] * inv + 1.0) * 1.5));
  const int b2 = min(2, (int)(((double)D[a2] * inv + 1.0) * 1.5));
  const double t = (0.5 * (double)(n[ax] * kCellUnits) - (double)O[ax]) / dax;
  const double N = (double)max(nx, max(ny, nz));
  const double scale = 64.0 / (3.0 * N * (double)kCellUnits);
  const double p1 = ((double)O[a1] + t * (double)D[a1] + N * kCellUnits) * scale;
  const double p2 = ((double)O[a2] + t * (double)D[a2] + N * kCellUnits) * scale;
  const uint32_t q1 = (uint32_t)fmin(63.0, fmax(0.0, p1));
  const uint32_t q2 = (uint32_t)fmin(63.0, fmax(0.0, p2));
  const uint32_t dir = (uint32_t)((ax * 2 + (D[ax] > 0)) * 9 + b1 * 3 + b2);
  return dir * 4096u + (spread6(q1) | (spread6(q2) << 1));
}

// a = 1 - e^{-tau} for tau >= 0, two accuracy levels.
//   precision form: degree-5 Taylor polynomial of (1 - e^{-tau})/tau below
//     tau = 1/4 (truncation < 5e-8), 1 - 2^{-tau log2 e} above (<= 5e-7);
//   plain form (march_plain): the same series to tau^3 below tau = 1/32
//     (truncation < 1.3e-6), written in the exponent argument, and
//     1 - 2^{-tau log2 e} above (<= 1.5e-6 just above the switch, falling
//     as 1/tau).
// The exponent is folded into base 2 per segment, as the paper's listing
// folds 1/ln 2 into the per-volume scalar.
__device__ __forceinline__ float poly5(float tau) {
  float p = fmaf(tau, -1.0f / 720.0f, 1.0f / 120.0f);
  p = fmaf(tau, p, -1.0f / 24.0f);
  p = fmaf(tau, p, 1.0f / 6.0f);
  p = fmaf(tau, p, -0.5f);
  p = fmaf(tau, p, 1.0f);
  return tau * p;
}

// ------------------------------------------------------ fixed-point tallies
// The absorbed and emitted power of every cell, and the entering and escaped
// power of the balance, are kept as exact integers: kAccDigits digits of
// kAccBits bits, digit k worth 2^(kAccBits k + kAccLsb) W, each held in a
// 64-bit word whose upper bits take the carries of up to 2^35 additions
// until the words are normalised (after every launch).  A value is rounded to
// kAccSig significant bits (relative error below 2^-kAccSig), which then
// span at most two digits, and added with integer atomics; integer additions
// commute, so every tally comes out the same bit for bit whatever order the
// wavefronts deliver their sums in.  Values below 2^kAccLsb W are dropped
// (truncation, the same in every order); a value that is NaN, negative or
// not below 2^80 W sets the overflow flag instead.
constexpr int kAccSig = kAccBits + 1;
static_assert(kAccSig + kAccBits - 1 <= 2 * kAccBits, "a rounded value spans two digits");
static_assert((80 - kAccSig - kAccLsb) / kAccBits + 1 <= kAccDigits - 1, "values below 2^80 W fit");
constexpr unsigned long long kAccMask = (1ull << kAccBits) - 1;

__device__ __forceinline__ void acc_add(unsigned long long* d, double v, unsigned* ovf) {
  if (!(v >= 0.0 && v < 0x1p80)) {
    atomicOr(ovf, 1u);
    return;
  }
  // v = mant 2^e, 1/2 <= mant < 1, e <= 80 (0 gives 0 and adds nothing); the
  // hardware frexp and 32-bit conversion, without the library's special cases
  int e = __builtin_amdgcn_frexp_exp(v);
  unsigned m = (unsigned)rint(ldexp(__builtin_amdgcn_frexp_mant(v), kAccSig));
  const unsigned up = m >> kAccSig;  // rounded up to 2^kAccSig
  m >>= up;
  e += (int)up;
  int p = e - kAccSig - kAccLsb;     // accumulator bit of m's lowest bit
  if (p < 0) {                       // partly or wholly below the lowest digit
    m = p <= -kAccSig ? 0u : m >> -p;
    p = 0;
  }
  if (m == 0) return;
  const unsigned k = (unsigned)p / kAccBits, s = (unsigned)p % kAccBits;
  const unsigned long long w = (unsigned long long)m << s;  // below 2^(2 kAccBits): digits k, k + 1
  atomicAdd(d + k, w & kAccMask);
  const unsigned long long hi = w >> kAccBits;
  if (hi) atomicAdd(d + k + 1, hi);
}

// Carries every digit's upper bits into the next digit.
__device__ __forceinline__ void acc_normalize(unsigned long long* d) {
  unsigned long long carry = 0;
#pragma unroll
  for (int k = 0; k < kAccDigits - 1; ++k) {
    const unsigned long long s = d[k] + carry;
    d[k] = s & kAccMask;
    carry = s >> kAccBits;
  }
  d[kAccDigits - 1] += carry;
}

// Digit sums of the copies (rows row, row + step, ...) of one accumulator
// row, normalised: the exact sum of the copies.
__device__ __forceinline__ void acc_sum_copies(const unsigned long long* acc, int64_t row,
                                               int64_t step, int copies,
                                               unsigned long long* d) {
#pragma unroll
  for (int k = 0; k < kAccRow; ++k) d[k] = 0;
  for (int r = 0; r < copies; ++r)
#pragma unroll
    for (int k = 0; k < kAccRow; ++k) d[k] += acc[(row + r * step) * kAccRow + k];
  acc_normalize(d);
  acc_normalize(d + kAccDigits);
}

// The value of normalised digits, summed from the top digit down.
__device__ __forceinline__ double acc_value(const unsigned long long* d) {
  double v = 0.0;
#pragma unroll
  for (int k = kAccDigits - 1; k >= 0; --k) v += ldexp((double)d[k], kAccBits * k + kAccLsb);
  return v;
}

// --------------------------------------------------------------- the march
// One wavefront, one ray, one spectral chunk: Eq. (3) cell after cell for
// every point, I <- I - (I - B) a with a = 1 - e^{-tau}.  Per segment every
// lane's partial sums of the chunk's absorbed (sum I a) and emitted (sum B a)
// radiance are staged in LDS; several segments at a time they are summed
// across the wavefront in a fixed order, weighted and added to the cells'
// fixed-point accumulators.  The ray's entering and escaped radiance over the
// chunk go the same way to the balance row.
//
// The plain form (march_plain) takes kPlainQ contiguous points per lane, the
// precision form (march_prec) 8 or 4, Planck values from the table, the degree-5
// branch and FP64 partial sums.
struct MarchWave {
  const float* kappa;   // row c at kappa + c * ld, column j - col0
  const float* planck;  // same layout (precision form)
  int64_t ld;
  int64_t col0;
  const double* theta;  // c2 / T per cell (plain form, general Planck values)
  const float4* poly;   // Planck cubics (plain form): record c * n_poly + chunk
  int64_t n_poly;
  const float* bwall;   // B(nu_j, T_wall), indexed by absolute j
  double nu0, dnu, c1, weight;
  unsigned long long* acc;  // accumulator rows, kAccRow words each
  int64_t row0;             // row of cell 0
  // copies of the cells' rows, rep_rows apart (a power of two of them): a ray
  // adds to copy (its slot & rep_mask), see acc_copies
  int64_t rep_rows;
  int rep_mask;
  int64_t bal_row0;         // first of the balance rows (entering, escaped)
  int bal_mask;             // balance rows - 1 (a power of two): a ray adds to
                            // row bal_row0 + (its slot & bal_mask)
  unsigned* ovf;            // set by acc_add for a value out of range
};

// Planck values of the plain form as one cubic per (cell, kMarchPoints-point
// chunk), B(nu_j, T) = r.x + r.y u + r.z u^2 + r.w u^3 with u = j minus the
// chunk's middle in points.  The host allows it (rt::planck_cubic_fits) where
// the cubic through the Chebyshev nodes and its first-order expansion over a
// lane's points are both within FP32 rounding of B; elsewhere a lane forms
// its own value (planck_lane).
constexpr int kMarchPoints = 64 * kPlainQ;
constexpr double kCubicNodeA = 0.92387953251128674, kCubicNodeB = 0.38268343236508978;

// Cubic through values at the nodes -a, -b, b, a of [-1, 1], for an argument
// in points (half = points per unit).
__host__ __device__ inline void planck_cubic(const double f[4], double half, double r[4]) {
  const double a = kCubicNodeA, b = kCubicNodeB, den = a * a - b * b;
  const double ea = 0.5 * (f[3] + f[0]), eb = 0.5 * (f[2] + f[1]);
  const double oa = 0.5 * (f[3] - f[0]) / a, ob = 0.5 * (f[2] - f[1]) / b;
  const double k2 = (ea - eb) / den, k3 = (oa - ob) / den;
  r[0] = ea - k2 * a * a;
  r[1] = (oa - k3 * a * a) / half;
  r[2] = k2 / (half * half);
  r[3] = k3 / (half * half * half);
}

// Per-wavefront LDS staging of the precision form's per-segment partial sums:
// [kSegs][64], even entries absorbed, odd emitted, each over a pair of lanes.
struct PrecStage {
  static constexpr int kSegs = 8;
  static constexpr int kEntries = kSegs * 64;
};

__device__ __forceinline__ void prec_stage(double* stage, int np, int lane, double ab, double em) {
  const double a2 = ab + dpp_f64<0xB1>(ab);  // quad_perm [1,0,3,2]
  const double e2 = em + dpp_f64<0xB1>(em);
  stage[np * 64 + lane] = (lane & 1) ? e2 : a2;
}

// Adds np staged entries to the accumulators.  Entry s is segment k0 + s of
// the ray, or the ray's balance row bal_row once k0 + s reaches ns.  Eight
// lanes per entry, each over 8 consecutive doubles (4 absorbed or entering, 4
// emitted or escaped), then across the eight with DPP: the same order every
// time.
__device__ __forceinline__ void prec_flush(const MarchWave& a, const double* stage,
                                           const int2* sg, int ns, int k0, int np, int lane,
                                           int64_t row0, int64_t bal_row) {
  static_assert(PrecStage::kSegs == 8, "flush layout");
  __builtin_amdgcn_wave_barrier();
  // a flush runs once per kSegs segments: its lane-derived addresses are
  // formed here rather than hoisted and kept live across the march loop
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int seg = ln >> 3, part = ln & 7;
  const double* src = stage + ln * 8;
  double s0 = src[0], s1 = src[1];
#pragma unroll
  for (int i = 2; i < 8; i += 2) {
    s0 += src[i];
    s1 += src[i + 1];
  }
  s0 += dpp_f64<0xB1>(s0);   // quad_perm [1,0,3,2]
  s1 += dpp_f64<0xB1>(s1);
  s0 += dpp_f64<0x4E>(s0);   // quad_perm [2,3,0,1]
  s1 += dpp_f64<0x4E>(s1);
  s0 += dpp_f64<0x141>(s0);  // row_half_mirror: the two quads of 8 lanes
  s1 += dpp_f64<0x141>(s1);
  __builtin_amdgcn_wave_barrier();
  if (part < 2 && seg < np) {
    const int k = k0 + seg;
    const int64_t row = k < ns ? row0 + sg[k].x : bal_row;
    acc_add(a.acc + row * kAccRow + part * kAccDigits, (part ? s1 : s0) * a.weight, a.ovf);
  }
}

// Wave-uniform loads through the scalar cache: for data that no block of the
// same launch writes (the persistent batched kernel, whose blocks write each
// other's segments, loads the ordinary way and broadcasts).
typedef int IntPair __attribute__((ext_vector_type(2)));
typedef float FloatQuad __attribute__((ext_vector_type(4)));
template <bool SCALAR>
__device__ __forceinline__ IntPair load_seg(const int2* p) {
  if (SCALAR)
    return *reinterpret_cast<const __attribute__((address_space(4))) IntPair*>(
        reinterpret_cast<uintptr_t>(p));
  const int2 v = *p;
  return IntPair{__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y)};
}
__device__ __forceinline__ FloatQuad load_quad(const float4* p) {
  return *reinterpret_cast<const __attribute__((address_space(4))) FloatQuad*>(
      reinterpret_cast<uintptr_t>(p));
}

// Precision form: points [j0, j0 + 64 Q) of one ray, j0 the same for the wave.
// stage: this wavefront's PrecStage::kEntries LDS entries; slot: the ray's
// index in its launch, which picks its balance row.
//
// A point takes 20 instructions and 8 bytes of the tables, a segment 40 more.
// Where rays share their cells' rows the instructions bound it and Q = 8 is
// taken: 24 points per lane left 8^3 cells too few wavefronts (1024 rays of
// 10,000 points 134 -> 111 us, 4096 rays 300 -> 247).  Where they do not, the
// rows come from beyond L2 at its rate, 7.4 TB/s, and what counts is how much
// of the launch's current chunk the caches hold: Q = 4 halves that chunk (24^3
// cells, 16,384 rays of 20,000 points: Q = 24 8.85 ms, 8 8.48, 4 7.99; 28^3,
// 65,536 rays 38.6, 38.1, 32.3).
template <bool EXIT, int Q>
__device__ __forceinline__ void march_prec(const MarchWave& a, const int2* sg, int ns, int64_t j0,
                                           int lane, float* exit_row, double* stage, int64_t slot) {
  constexpr int kSegs = PrecStage::kSegs;
  const int64_t row0 = a.row0 + (slot & a.rep_mask) * a.rep_rows;
  float I[Q];
#pragma unroll
  for (int h = 0; h < Q / 4; ++h) {
    const float4 v = *reinterpret_cast<const float4*>(a.bwall + j0 + lane * Q + 4 * h);
    I[4 * h] = v.x; I[4 * h + 1] = v.y; I[4 * h + 2] = v.z; I[4 * h + 3] = v.w;
  }
  double enter = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) enter += (double)I[q];
  const float nlog2e = -1.4426950408889634f;
  int np = 0, k0 = 0;  // staged entries, and the segment of the first
  IntPair s = ns > 0 ? load_seg<true>(sg) : IntPair{0, 0};
  const unsigned voff = (unsigned)lane * (4 * Q);
  const char* kchunk = reinterpret_cast<const char*>(a.kappa + j0 - a.col0);
  const char* pchunk = reinterpret_cast<const char*>(a.planck + j0 - a.col0);
  for (int k = 0; k < ns; ++k) {
    const int64_t c = s.x;
    const float l = __int_as_float(s.y);
    const float xs = l * nlog2e;
    float kv[Q], bv[Q];
    const char* krow = kchunk + c * (a.ld * 4);
    const char* prow = pchunk + c * (a.ld * 4);
    unsigned vo = voff;  // opaque: the rows' addresses stay uniform, not per lane
    asm("" : "+v"(vo));
#pragma unroll
    for (int h = 0; h < Q / 4; ++h) {
      const float4 v = *reinterpret_cast<const float4*>(krow + vo + 16 * h);
      kv[4 * h] = v.x; kv[4 * h + 1] = v.y; kv[4 * h + 2] = v.z; kv[4 * h + 3] = v.w;
    }
#pragma unroll
    for (int h = 0; h < Q / 4; ++h) {
      const float4 v = *reinterpret_cast<const float4*>(prow + vo + 16 * h);
      bv[4 * h] = v.x; bv[4 * h + 1] = v.y; bv[4 * h + 2] = v.z; bv[4 * h + 3] = v.w;
    }
    if (k + 1 < ns) s = load_seg<true>(sg + k + 1);  // the next segment's, early
    // a = 1 - e^{-tau} per point
    float av[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float tau = kv[q] * l;
      const float big = 1.0f - __builtin_amdgcn_exp2f(kv[q] * xs);
      av[q] = tau < 0.25f ? poly5(tau) : big;
    }
    double ab = 0, em = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      ab += (double)(I[q] * av[q]);
      em += (double)(bv[q] * av[q]);
      I[q] = fmaf(-(I[q] - bv[q]), av[q], I[q]);
    }
    // the update of I is complete here, so a[] dies before the staging and
    // the flush below (the scheduler would otherwise sink the updates past
    // them and keep a[] and B[] live across the flush)
#pragma unroll
    for (int q = 0; q < Q; ++q) asm volatile("" ::"v"(I[q]));
    prec_stage(stage, np, lane, ab, em);
    if (++np == kSegs) {
      prec_flush(a, stage, sg, ns, k0, np, lane, row0, 0);
      k0 += np;
      np = 0;
    }
  }
  double esc = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) esc += (double)I[q];
  if (EXIT) {
#pragma unroll
    for (int h = 0; h < Q / 4; ++h)
      *reinterpret_cast<float4*>(exit_row + j0 - a.col0 + lane * Q + 4 * h) =
          make_float4(I[4 * h], I[4 * h + 1], I[4 * h + 2], I[4 * h + 3]);
  }
  // np < kSegs here: one more entry, the balance row's (entering, escaped)
  prec_stage(stage, np, lane, enter, esc);
  prec_flush(a, stage, sg, ns, k0, np + 1, lane, row0, a.bal_row0 + (slot & a.bal_mask));
}

// ------------------------------------------------------- the plain form's march
// Staging of the plain form: one float per lane and segment.  Lanes 2 i and
// 2 i + 1 hold the pair's absorbed and emitted sums (one DPP add each and a
// select), so 16 segments take the 4 KB that 8 took unpaired, and a flush,
// whose cost is the fixed-point add whatever it carries, runs half as often.
struct PlainStage {
  static constexpr int kSegs = 16;
  static constexpr int kEntries = kSegs * 64;
};

__device__ __forceinline__ void plain_stage(float* stage, int np, int lane, float ab, float em) {
  const float a2 = ab + dpp_f32<0xB1>(ab);  // quad_perm [1,0,3,2]
  const float e2 = em + dpp_f32<0xB1>(em);
  stage[np * 64 + lane] = (lane & 1) ? e2 : a2;
}

// Adds np staged entries to the accumulators (entries as prec_flush).  Four
// lanes per entry, each over 16 consecutive floats (8 absorbed, 8 emitted),
// then across the four with DPP: the same order every time.
__device__ __forceinline__ void plain_flush(const MarchWave& a, const float* stage, const int2* sg,
                                            int ns, int k0, int np, int lane, int64_t row0,
                                            int64_t bal_row) {
  __builtin_amdgcn_wave_barrier();
  int ln = lane;  // see prec_flush
  asm volatile("" : "+v"(ln));
  const int seg = ln >> 2;
  const float4* src = reinterpret_cast<const float4*>(stage + ln * 16);
  float ab = 0.f, em = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float4 v = src[i];
    ab += v.x;
    em += v.y;
    ab += v.z;
    em += v.w;
  }
  ab += dpp_f32<0xB1>(ab);
  em += dpp_f32<0xB1>(em);
  float s = (ln & 1) ? em : ab;
  s += dpp_f32<0x4E>(s);  // quad_perm [2,3,0,1]
  __builtin_amdgcn_wave_barrier();
  if (!(ln & 2) && seg < np) {
    const int k = k0 + seg;
    const int64_t row = k < ns ? row0 + sg[k].x : bal_row;
    acc_add(a.acc + row * kAccRow + (ln & 1) * kAccDigits, (double)s * a.weight, a.ovf);
  }
}

// General Planck values of a lane (plain form, where the cubics do not fit):
// one exact value at its first point nu_a and the second-order expansion of
// ln B:
//   B(nu_a + d) = B_a (1 + g1 d + (g1^2 + g2) d^2 / 2),
//   g1 = 3/nu - theta (1 + r),  g2 = -3/nu^2 + theta^2 r (1 + r),
//   theta = c2 / T,  r = 1 / (exp(theta nu) - 1).
struct PlanckLane {
  double nu_a;
  float c1nu3, three_nu, three_nu2, dnu;
};
__device__ __forceinline__ void planck_lane(const PlanckLane& p, double th, float& B0, float& K1,
                                            float& K2) {
  // exp(theta nu_a) with FP64 range reduction: 2^n 2^f, |f| <= 1/2
  const double z = th * 1.4426950408889634074 * p.nu_a;
  const double n = rint(z);
  const float f = (float)(z - n);
  const float e = ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
  float em1 = e - 1.0f;
  if (__ballot(z < 0.36)) {  // theta nu < 1/4: expm1 by its series
    const float x = (float)(th * p.nu_a);
    float q = fmaf(x, 1.0f / 720.0f, 1.0f / 120.0f);
    q = fmaf(x, q, 1.0f / 24.0f);
    q = fmaf(x, q, 1.0f / 6.0f);
    q = fmaf(x, q, 0.5f);
    q = fmaf(x, q, 1.0f);
    if (z < 0.36) em1 = x * q;
  }
  const float r = __builtin_amdgcn_rcpf(em1);
  B0 = p.c1nu3 * r;
  const float thf = (float)th;
  const float t1 = 1.0f + r;
  const float g1 = fmaf(-thf, t1, p.three_nu);
  const float g2 = fmaf(thf * thf, r * t1, -p.three_nu2);
  K1 = B0 * g1 * p.dnu;
  K2 = 0.5f * B0 * fmaf(g1, g1, g2) * (p.dnu * p.dnu);
}

// One wavefront, one ray, the kMarchPoints points from the absolute index j0
// (uniform), kPlainQ per lane.
//
// Issue-bound where rays are dense: a point takes its multiply, the
// exponential, a, B, I - B, the update, two sums and half a maximum, 8.5
// instructions, and a segment 26 more (Planck cubic, test, staging, flush, the
// ray's ends), shared by the lane's kPlainQ points.  24 points per lane spread
// those best but put 6 KB of each crossed cell's row in flight per wavefront, a
// whole XCD's L2.  32^3 cells, 50,000 points, 2^20 rays: 10.7 instructions per
// update and 2.6 TB past L2 in 505 to 512 ms at 12 points (at 24 points with
// general Planck values, the result copied around the loop, it was 11.6
// instructions, 3.45 TB and 562 ms).  Where rays are sparse (about 100 per cell)
// each row is read from beyond L2 for nearly every crossing, at 7 TB/s, and fewer
// wavefronts in flight are better: the launches pad the block's LDS to hold 6 or 7
// per SIMD.
//
// Both the sums and the update of I take a and not e^-tau: sums of I e^-tau and
// (I - B) e^-tau + B save an instruction a point and lose a thin cell's a, and
// with it what the cells behind absorb and the walls receive (cold walls, 16
// cells of tau = 1e-4: 2e-4 of the absorbed power).  a is tau - tau^2/2 +
// tau^3/6, written in x = -tau log2(e) (truncation below tau^3/24 = 1.3e-6
// relative), below tau = 1/32 and 1 - e^-tau from there on; a wavefront without
// a thinner point skips the series.
// CUBIC: Planck cubics, else planck_lane.  SCALAR: see load_seg.
// stage: this wavefront's PlainStage::kEntries LDS floats; slot: the ray's
// index in its launch, which picks its balance row.
template <bool EXIT, bool CUBIC, bool SCALAR>
__device__ __forceinline__ void march_plain(const MarchWave& a, const int2* sg, int ns, int64_t j0,
                                            int lane, float* exit_row, float* stage,
                                            int64_t slot) {
  constexpr int Q = kPlainQ;
  const int64_t row0 = a.row0 + (slot & a.rep_mask) * a.rep_rows;
  constexpr float nlog2e = -1.4426950408889634f;
  constexpr float kThinX = 0.03125f * nlog2e;  // tau = 1/32
  const unsigned voff = (unsigned)lane * (Q * 4);            // bytes into the chunk's row
  const char* kchunk = reinterpret_cast<const char*>(a.kappa + (j0 - a.col0));
  const int64_t j = j0 + lane * Q;
  float I[Q];
#pragma unroll
  for (int h = 0; h < Q / 4; ++h) {
    const float4 v = *reinterpret_cast<const float4*>(a.bwall + j + 4 * h);
    I[4 * h] = v.x; I[4 * h + 1] = v.y; I[4 * h + 2] = v.z; I[4 * h + 3] = v.w;
  }
  const float4* poly = nullptr;
  float u0 = 0.f;  // the lane's first point from the chunk's middle
  PlanckLane pl{};
  if (CUBIC) {
    poly = a.poly + j0 / kMarchPoints;
    u0 = (float)(lane * Q) - 0.5f * (kMarchPoints - 1);
  } else {
    pl.nu_a = a.nu0 + (double)j * a.dnu;
    pl.c1nu3 = (float)(a.c1 * pl.nu_a * pl.nu_a * pl.nu_a);
    pl.three_nu = (float)(3.0 / pl.nu_a);
    pl.three_nu2 = (float)(3.0 / (pl.nu_a * pl.nu_a));
    pl.dnu = (float)a.dnu;
  }
  float enter = 0.f;
#pragma unroll
  for (int q = 0; q < Q; ++q) enter += I[q];
  int np = 0, k0 = 0;  // staged entries, and the segment of the first
  IntPair s = ns > 0 ? load_seg<SCALAR>(sg) : IntPair{0, 0};
  for (int k = 0; k < ns; ++k) {
    const int64_t c = s.x;
    const float l = __int_as_float(s.y);
    FloatQuad r{};
    if (CUBIC) r = load_quad(poly + c * a.n_poly);
    float kv[Q];
    {
      const char* row = kchunk + c * (a.ld * 4);
      unsigned vo = voff;  // opaque: the row's address stays uniform, not per lane
      asm("" : "+v"(vo));
#pragma unroll
      for (int h = 0; h < Q / 4; ++h) {
        const float4 v = *reinterpret_cast<const float4*>(row + vo + 16 * h);
        kv[4 * h] = v.x; kv[4 * h + 1] = v.y; kv[4 * h + 2] = v.z; kv[4 * h + 3] = v.w;
      }
    }
    s = load_seg<SCALAR>(sg + min(k + 1, ns - 1));  // the next segment's, early
    const float xs = l * nlog2e;
    float B0, K1, K2 = 0.f;
    if (CUBIC) {
      const float e2 = fmaf(r.w, u0, r.z);
      const float e1 = fmaf(e2, u0, r.y);
      B0 = fmaf(e1, u0, r.x);
      K1 = fmaf(fmaf(r.w, u0, e2), u0, e1);  // the derivative at u0
    } else {
      planck_lane(pl, a.theta[c], B0, K1, K2);
    }
    asm("" : "+v"(B0), "+v"(K1));  // formed here: their load is not put off past the test
    float av[Q], B[Q];  // a, and x until the series have been chosen
    float xmax = kv[0] * xs;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float x = kv[q] * xs;
      xmax = fmaxf(xmax, x);
      av[q] = 1.0f - __builtin_amdgcn_exp2f(x);
      B[q] = q == 0 ? B0 : fmaf(CUBIC ? K1 : fmaf(K2, (float)q, K1), (float)q, B0);
    }
    if (__ballot(xmax > kThinX)) {
      constexpr float L1 = -0.69314718055994531f, L2 = -0.24022650695910071f,
                      L3 = -0.055504108664821576f;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float x = kv[q] * xs;
        const float ser = x * fmaf(x, fmaf(x, L3, L2), L1);
        av[q] = x > kThinX ? ser : av[q];
      }
    }
    float ab2[2] = {0.f, 0.f}, em2[2] = {0.f, 0.f};  // two chains: half the roundings in a row
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      ab2[q & 1] = fmaf(I[q], av[q], ab2[q & 1]);
      em2[q & 1] = fmaf(B[q], av[q], em2[q & 1]);
      // I <- I - (I - B) a, in place: the compiler would form it beside I, keep
      // a and B live across the flush and copy the Q results back around the loop
      asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(I[q]) : "v"(B[q] - I[q]), "v"(av[q]));
    }
    plain_stage(stage, np, lane, ab2[0] + ab2[1], em2[0] + em2[1]);
    if (++np == PlainStage::kSegs) {
      plain_flush(a, stage, sg, ns, k0, np, lane, row0, 0);
      k0 += np;
      np = 0;
    }
  }
  float esc = 0.f;
#pragma unroll
  for (int q = 0; q < Q; ++q) esc += I[q];
  if (EXIT) {
#pragma unroll
    for (int h = 0; h < Q / 4; ++h)
      *reinterpret_cast<float4*>(exit_row + (j - a.col0) + 4 * h) =
          make_float4(I[4 * h], I[4 * h + 1], I[4 * h + 2], I[4 * h + 3]);
  }
  // np < kSegs here: one more entry, the balance row's (entering, escaped)
  plain_stage(stage, np, lane, enter, esc);
  plain_flush(a, stage, sg, ns, k0, np + 1, lane, row0, a.bal_row0 + (slot & a.bal_mask));
}

}  // namespace dev

// kappa.hip: the handle's walls' row; and, where the call writes no Planck table
// (whose launch has it), its place behind the `blocks` of a launch: the number of
// its blocks (else none)
dev::WallRow wall_row_of(rt_ctx c);
unsigned add_wall_row(rt_ctx c, dev::WallRow& w, int64_t blocks, int threads);

// Line-sum tiles [tile_begin, tile_begin + n_tiles) for n_cell_groups groups
// of kKappaCells cells (kappa.hip).
hipError_t launch_kappa_tiles(rt_ctx c, const dev::KappaTile& t, int64_t n_cell_groups,
                              int tile_begin, int n_tiles, bool comp, hipStream_t s,
                              const dev::TileGate& gate = dev::TileGate(), int parts = 1,
                              int64_t part_stride = 0);

}  // namespace rt
