// kappa.hip -- per-cell spectral properties on gfx950.
//
//   cell_params   : per-cell gas state -> FP32/FP64 factors (FP64 arithmetic)
//   kappa_linesum : Eq. (2) with the Eq. (1) strength ratio (line tiles staged
//                   in LDS, kappa written coalesced along nu): plain
//                   (dev::kappa_tile_far) and compensated (dev::kappa_tile,
//                   dev::kappa_tile_comp)
//   planck_table  : Eq. (4), wavenumber form, per (cell, nu) and for the walls,
//                   evaluated in FP32 (pair arguments, exp_pair/expm1_pair)
#include <cfloat>
#include <climits>

#include "batch_plan.h"
#include "device_common.h"
#include "launch_pieces.h"

namespace rt {
namespace {

using namespace dev;

// ---------------------------------------------------------------- cells
// u = x p / (k_B T) [cm^-3]; q = (T_ref/T)^1.5 (partition-function ratio of
// Eq. (1)); G = u q / (pi dnu) with energies, u / (pi dnu) without.
__device__ inline float cell_G(double T, double x, double p, double T_ref, double dnu,
                               int have_E) {
  const double u = x * p * kAtm / (kBoltzmann * T) * 1e-6;
  const double q = have_E ? pow(T_ref / T, 1.5) : 1.0;
  return (float)(u * q / (M_PI * dnu));
}

__global__ void cell_params_kernel(int64_t n, const double* __restrict__ T,
                                   const double* __restrict__ x,
                                   const double* __restrict__ p, double T_ref,
                                   double dnu, double c2, int have_E,
                                   float* G, double* beta, double* theta,
                                   float* lam2, float* P) {
  int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  double Tc = T[c];
  G[c] = cell_G(Tc, x[c], p[c], T_ref, dnu, have_E);
  beta[c] = 1.0 / T_ref - 1.0 / Tc;
  theta[c] = c2 / Tc;
  lam2[c] = (float)log2(T_ref / Tc);
  P[c] = (float)(p[c] / dnu);
}

// The plain line sum's records of a line list, from its arrays.
__global__ void line_data_kernel(LineSet L) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= L.n) return;
  L.data[i] = LineData{(float)L.m[i], L.phi[i], (float)(L.wlo[i] - L.m[i]), L.S[i], L.gamma[i],
                       L.nexp[i], 0.f, 0.f, L.E2[i], L.nu[i]};
}

// The precision form's Gq = u q / (pi dnu) per cell, in FP32: u/(pi dnu) and
// log2(T_ref/T) come from the host, q = 2^(1.5 log2(T_ref/T)) with energies
// (the partition ratio of Eq. (1)), 1 without.
__global__ void cell_params32_kernel(int64_t n, const float* __restrict__ uf,
                                     const float* __restrict__ lamf, int have_E, float* Gq) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  Gq[c] = have_E ? uf[c] * fast_exp2(1.5f * lamf[c]) : uf[c];
}

// G of a further gas: its own mole fraction and partition-ratio choice.
__global__ void gas_factor_kernel(int64_t n, const double* __restrict__ T,
                                  const double* __restrict__ x, const double* __restrict__ p,
                                  double T_ref, double dnu, int have_E, float* G) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  G[c] = cell_G(T[c], x[c], p[c], T_ref, dnu, have_E);
}

struct KappaArgs {
  KappaTile t;
  int n_tiles;
  int tile_begin;
  int64_t group0 = 0;        // the launch's first group of cells
  TileGate gate;
  int parts = 1;             // line shares per tile, each into its own output
  int64_t part_stride = 0;   // floats between the shares' outputs
  WallRow wall;              // plain form: its blocks follow the tiles'
};

// FORM: kPlainSum (P spans per wavefront), kCompSum (the batched launches'
// compensated sum, one span), kPrecSum (the precision form's).
constexpr int kPlainSum = 0, kCompSum = 1, kPrecSum = 2;
template <int FORM, int P>
__global__ __launch_bounds__(FORM == kPrecSum ? kPrecThreads : kKappaThreads)
__attribute__((amdgpu_waves_per_eu(FORM == kPrecSum ? 6 : 5))) void kappa_linesum_kernel(KappaArgs a) {
  static_assert(FORM != kCompSum || P == 1, "a span per wavefront");
  static_assert(FORM != kPrecSum || kKappaThreads * P == kPrecThreads, "kappa_tile's points");
  __shared__ float4 lds4[kLineTile * kLineRec / 4];
  __shared__ float4 fx4[FORM == kPrecSum ? 1 : kFarEntries];  // floats, or doubles, of 4 wavefronts
  auto sum_tile = [&](const KappaTile& t, int j0, int64_t cell0, bool on) {
    float* lds = reinterpret_cast<float*>(lds4);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (FORM == kPrecSum)
      kappa_tile(t, j0, cell0, lds);
    else if constexpr (FORM == kCompSum)
      kappa_tile_comp(t, j0, cell0, lds, reinterpret_cast<double*>(fx4) + wave * kCompEntries);
    else
      kappa_tile_far<P>(t, j0, cell0, lds, reinterpret_cast<float*>(fx4) + wave * kFarEntries, on);
  };
  if constexpr (FORM == kPlainSum) {
    if (blockIdx.x >= a.wall.first) {
      wall_row(a.wall, blockIdx.x - a.wall.first, kKappaThreads);
      return;
    }
  }
  const int part = (int)(blockIdx.x % (unsigned)a.parts);
  const int64_t tb = blockIdx.x / (unsigned)a.parts;
  const int tile = (int)(tb % a.n_tiles);
  const int64_t cg = a.group0 + tb / a.n_tiles;
  constexpr int kTilePoints = kKappaThreads * P;
  const int j0 = (a.tile_begin + tile) * kTilePoints;
  bool wave_on = true;
  if (a.gate.group_flag || a.gate.chunk_err) {
    const bool marked = a.gate.group_flag && a.gate.group_flag[cg] == a.gate.epoch;
    bool need = marked;
    if (a.gate.chunk_err) {
      const int c0 = j0 / a.gate.chunk_w;
      const int c1 = min(a.gate.n_chunks - 1, (j0 + kTilePoints - 1) / a.gate.chunk_w);
      for (int k = c0; k <= c1; ++k) need = need || a.gate.chunk_err[k] > a.gate.tol;
      // a wavefront's 64 P points lie in one chunk when chunks are a
      // multiple of that span: then only the wavefronts of chunks over
      // tolerance (or of marked cells) evaluate and write; the others only
      // help stage the line records
      constexpr int kSpan = 64 * P;
      if (!marked && a.gate.chunk_w % kSpan == 0) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int k = (j0 + wave * kSpan) / a.gate.chunk_w;
        wave_on = k < a.gate.n_chunks && a.gate.chunk_err[k] > a.gate.tol;
      }
    }
    if (!need) return;
  }
  if (a.parts > 1) {
    KappaTile t = a.t;
    t.line_parts = a.parts;
    t.line_part = part;
    t.out += part * a.part_stride;
    sum_tile(t, j0, cg * kKappaCells, wave_on);
    return;
  }
  sum_tile(a.t, j0, cg * kKappaCells, wave_on);
}

// Planck table: one block per (kPlanckCells cells, 256-point segment of their
// rows), so that a point's wavenumber and its cube serve several cells.
// Issue-bound; 16^3 cells, 20,000 points: 73 us (one cell per block: 175).  The
// walls' row follows the last cells'.
constexpr int kPlanckCells = 8;
__global__ __launch_bounds__(256) void planck_table_kernel(
    const float2* __restrict__ theta2, int64_t n_cells, int n_nu, int64_t ld, int tiles_per_row,
    float2 nu0, float2 dnu, float c1, float* __restrict__ B, WallRow wall) {
  const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t cell0 = b / tiles_per_row * kPlanckCells;
  const int64_t wall0 = (n_cells + kPlanckCells - 1) / kPlanckCells * tiles_per_row;
  if (b >= wall0) {  // (a grid of several rows of blocks has more than needed)
    wall_row(wall, b - wall0, 256);
    return;
  }
  const int64_t j = b % tiles_per_row * 256 + threadIdx.x;
  if (cell0 >= n_cells || j >= ld) return;
  const Pair nu = nu_at(j, pair_of(nu0), pair_of(dnu));
  const int cells = (int)min<int64_t>(kPlanckCells, n_cells - cell0);
  float* o = B + cell0 * ld + j;
  for (int k = 0; k < cells; ++k, o += ld)
    *o = j < n_nu ? planck_f32(nu, pair_of(theta2[cell0 + k]), c1) : 0.f;
}

// Planck cubics of the plain march: one thread per (cell, chunk of
// kMarchPoints points), B at the four Chebyshev nodes in FP64.
__global__ void planck_cubics_kernel(const double* __restrict__ theta, int64_t n, int64_t n_chunks,
                                     double nu0, double dnu, double c1,
                                     float4* __restrict__ poly) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * n_chunks) return;
  const double th = theta[i / n_chunks];
  const double half = 0.5 * kMarchPoints;
  const double mid = nu0 + ((double)(i % n_chunks) * kMarchPoints + 0.5 * (kMarchPoints - 1)) * dnu;
  const double x[4] = {-kCubicNodeA, -kCubicNodeB, kCubicNodeB, kCubicNodeA};
  double f[4], r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double nu = mid + x[k] * half * dnu;
    f[k] = c1 * nu * nu * nu / expm1(th * nu);
  }
  planck_cubic(f, half, r);
  poly[i] = make_float4((float)r[0], (float)r[1], (float)r[2], (float)r[3]);
}

// The paper's own formulation of Eq. (2) (Section 3 and its listing): line i
// contributes u S_i s_i(T) f_i(j) at the 16 grid points j = m_i - 7 .. m_i + 8,
// f_i the reference-state Lorentz shape tabulated once per line (prof16);
// u S s is the plain line sum's amplitude without the half width (G pi dnu S
// and the Eq. (1) factors).
//
// kappa = (cells x lines amplitudes) (lines x points profiles): a banded
// product, done with v_mfma_f32_32x32x2_f32, two lines a step, on tiles of 32
// cells x 32 points.  One block per (64 cells, 256 points), each of its eight
// wavefronts owning 32 points of both 32-cell halves, which share the profile
// operand; the lines whose 16 points meet the block's points (tile16, found
// once per line list) are staged in LDS 64 at a time: m, the 16 values with a
// zero behind them, which every point outside the 16 reads, and the
// amplitudes of the 64 cells, lane = cell, so that a line's inputs are scalar
// loads.  32 points wide, a tile meets the lines of 47 points, so a third of
// the products are real ones; a tile of 64 points would have a fifth, and
// 16-point tiles twice the LDS reads per product.  All gases add into one set of
// accumulators, so a row is written once.
// 32^3 cells, 50,000 points, 20,000 lines: 1.7 ms, of which writing the 6.6 GB
// is 1.0, the amplitudes' instructions 0.8 and the matrix instructions 0.45
// (8 cells per thread and a multiply-add per point and line of its 64 points
// took 4.1).  The stores bypass the caches: with ordinary ones 2.1 ms.  Two
// gases in a launch each, that adds to the rows, and in one: 5,850 cells, 8,297
// points, 12 lines per cm^-1 172, 53 us; 16^3 cells, 20,000 points 278, 96.
constexpr int kT16Points = 256;
constexpr int kT16Cells = 64;
constexpr int kT16Stage = 64;
constexpr int kT16Threads = 2 * kT16Points;
typedef float f32x16 __attribute__((ext_vector_type(16)));
// the cell row of register i of a lane in the first lane half (rows 4 further in the second)
__device__ constexpr int t16_row(int i) { return (i & 3) + 8 * (i >> 2); }
template <class T>
__device__ __forceinline__ T load_const(const T* p) {  // a wave's same address: a scalar load
  return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}
struct T16Gas {
  const int2* tile16;
  const LineData* data;
  const float* prof16;
  const int* m;
  const float* G;
  int n_tiles16, have_E;
};
struct T16Gases {
  T16Gas g[kMaxGases];
  int n;
};
__global__ __launch_bounds__(kT16Threads) __attribute__((amdgpu_waves_per_eu(6))) void kappa_table16_kernel(
    T16Gases gases, const double* __restrict__ beta_, const double* __restrict__ theta_,
    int64_t n_cells, int n_nu, int64_t ld, int n_tiles, double pi_dnu, float* __restrict__ out,
    WallRow wall) {
  if (blockIdx.x >= wall.first) {
    wall_row(wall, blockIdx.x - wall.first, kT16Threads);
    return;
  }
  // one row more than staged lines: a pair's second line past the last one
  __shared__ int s_m[kT16Stage + 1];
  __shared__ float s_tab[(kT16Stage + 1) * 17];
  __shared__ float s_amp[(kT16Stage + 1) * kT16Cells];
  const int tile = blockIdx.x % n_tiles;
  const int64_t cell0 = (int64_t)(blockIdx.x / n_tiles) * kT16Cells;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, sub = lane & 31;
  const int wj = tile * kT16Points + 32 * wave;
  const int64_t own = min(cell0 + lane, n_cells - 1);
  const double beta = beta_[own], theta = theta_[own];
  auto lines_of = [&](const T16Gas& g) {  // those whose 16 points meet the block's
    return tile < g.n_tiles16 ? g.tile16[tile] : make_int2(0, 0);
  };
  auto factor_of = [&](const T16Gas& g) { return (float)((double)g.G[own] * pi_dnu); };
  auto amplitude = [&](const T16Gas& g, float G, int i) {
    const LineData* d = g.data + i;
    float amp = G * load_const(&d->S);
    if (g.have_E) {
      amp *= exp_split(load_const(&d->E2) * beta);
      amp *= one_minus_exp_neg_d(load_const(&d->nu) * theta);
    }
    return amp;
  };
  bool over = false;  // an amplitude beyond float: its line is left to the end
  f32x16 acc[2] = {};  // [cell half]
  for (int k = 0; k < gases.n; ++k) {
    const T16Gas& g = gases.g[k];
    const int2 range = lines_of(g);
    const float G = factor_of(g);
    for (int base = range.x; base < range.y; base += kT16Stage) {
      const int nt = min(kT16Stage, range.y - base);
      __syncthreads();
#pragma unroll 2
      for (int li = wave; li < nt; li += kT16Threads / 64) {
        const float amp = amplitude(g, G, base + li);
        const bool fits = fabsf(amp) <= FLT_MAX;
        over |= !fits;
        s_amp[li * kT16Cells + lane] = fits ? amp : 0.f;
      }
      for (int q = tid; q < nt * 16; q += kT16Threads)
        s_tab[(q >> 4) * 17 + (q & 15)] = g.prof16[(int64_t)base * 16 + q];
      int m = INT_MAX / 2;  // a lane's staged line
      if (lane < nt) m = g.m[base + lane];
      if (wave == 0) {
        s_m[lane] = m;
        s_tab[lane * 17 + 16] = 0.f;
      } else if (wave == 1) {  // the row behind the last line
        s_amp[nt * kT16Cells + lane] = 0.f;
        if (lane < 17) s_tab[nt * 17 + lane] = 0.f;
        if (lane == 0) s_m[kT16Stage] = INT_MAX / 2;
      }
      __syncthreads();
      // the staged lines meeting the tile's points: m in [wj - 8, wj + 31 + 7]
      const int l0 = __popcll(__ballot(m < wj - 8)), l1 = __popcll(__ballot(m <= wj + 38));
      const int jt = wj + sub + 7;
      for (int l = l0; l < l1; l += 2) {
        const int li = l + half;
        const unsigned u = min((unsigned)(jt - s_m[li]), 16u);
        const float f = s_tab[li * 17 + u];
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(s_amp[li * kT16Cells + sub], f, acc[0], 0, 0, 0);
        acc[1] =
            __builtin_amdgcn_mfma_f32_32x32x2f32(s_amp[li * kT16Cells + 32 + sub], f, acc[1], 0, 0, 0);
      }
    }
  }
  if (wj < ld) {
    const unsigned off = 4 * half * (unsigned)ld + sub;  // ld < 2^25
    if (cell0 + kT16Cells <= n_cells && wj + 32 <= n_nu) {
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        float* o = out + (cell0 + t16_row(i)) * ld + wj;
        __builtin_nontemporal_store(acc[i >> 4][i & 15], o + off);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const int64_t cell = cell0 + t16_row(i);
        if (cell + 4 * half >= n_cells) continue;
        float* o = out + cell * ld + wj;
        __builtin_nontemporal_store(wj + sub < n_nu ? acc[i >> 4][i & 15] : 0.f, o + off);
      }
    }
  }
  // Zeros of the band times an infinite amplitude would be NaN: such lines add
  // to their own 16 points only.  One wavefront, a lane per row.
  if (__syncthreads_or(over) && wave == 0 && cell0 + lane < n_cells) {
    for (int k = 0; k < gases.n; ++k) {
      const T16Gas& g = gases.g[k];
      const int2 range = lines_of(g);
      const float G = factor_of(g);
      for (int i = range.x; i < range.y; ++i) {
        const float amp = amplitude(g, G, i);
        if (fabsf(amp) <= FLT_MAX) continue;
        for (int t = 0; t < 16; ++t) {
          const int j = g.m[i] - 7 + t;
          if (j >= tile * kT16Points && j < min((tile + 1) * kT16Points, n_nu))
            out[own * ld + j] = fmaf(amp, g.prof16[(int64_t)i * 16 + t], out[own * ld + j]);
        }
      }
    }
  }
}

}  // namespace

// v as an FP32 pair hi + lo (host).
static float2 host_pair(double v) {
  const float h = (float)v;
  return make_float2(h, (float)(v - (double)h));
}

dev::WallRow wall_row_of(rt_ctx c) {
  dev::WallRow w;
  w.theta = c->T_wall > 0.0 ? host_pair(second_radiation_cm_K() / c->T_wall) : make_float2(0.f, 0.f);
  w.nu0 = host_pair(c->nu0);
  w.dnu = host_pair(c->dnu);
  w.c1 = (float)first_radiation_wavenumber();
  w.n_nu = c->n_nu;
  w.ld = c->ld;  // a multiple of 1536: whole blocks of 256 or 512
  w.out = c->d_bwall;
  return w;
}

unsigned add_wall_row(rt_ctx c, dev::WallRow& w, int64_t blocks, int threads) {
  if (c->planck) return 0;
  w = wall_row_of(c);
  w.first = (unsigned)blocks;
  return (unsigned)(c->ld / threads);
}

hipError_t launch_kappa_table16(rt_ctx c) {
  const int n_tiles = (int)((c->ld + kT16Points - 1) / kT16Points);
  const int64_t blocks = (c->n_cells + kT16Cells - 1) / kT16Cells * n_tiles;
  if (!launch_fits(blocks + c->ld / kT16Threads, kT16Threads)) return hipErrorInvalidValue;
  T16Gases gases{};
  auto add = [&](const LineSet& L, const float* G, bool have_E) {
    gases.g[gases.n++] = T16Gas{L.tile16, L.data, L.prof16, L.m, G, L.n_tiles16, have_E ? 1 : 0};
  };
  add(c->lines, c->cells.G, c->have_E);
  for (const auto& gs : c->gas)
    if (gs.active) add(gs.lines, gs.G, gs.have_E);
  dev::WallRow wall;
  const unsigned walls = add_wall_row(c, wall, blocks, kT16Threads);
  hipLaunchKernelGGL(kappa_table16_kernel, dim3((unsigned)blocks + walls), dim3(kT16Threads), 0,
                     c->stream, gases, c->cells.beta, c->cells.theta, c->n_cells, c->n_nu, c->ld,
                     n_tiles, M_PI * c->dnu, c->kappa, wall);
  return hipGetLastError();
}

hipError_t launch_line_data(rt_ctx c, const LineSet& L) {
  if (L.n > 0)
    hipLaunchKernelGGL(line_data_kernel, dim3((unsigned)((L.n + 255) / 256)), dim3(256), 0,
                       c->stream, L);
  return hipGetLastError();
}

hipError_t launch_cell_params(rt_ctx c) {
  const int64_t n = c->n_cells;
  const int threads = 256;
  const int64_t blocks = (n + threads - 1) / threads;
  hipLaunchKernelGGL(cell_params_kernel, dim3((unsigned)blocks), dim3(threads), 0, c->stream,
                     n, c->d_T, c->d_x, c->d_p, c->T_ref, c->dnu, second_radiation_cm_K(),
                     c->have_E ? 1 : 0, c->cells.G, c->cells.beta, c->cells.theta,
                     c->cells.lam2, c->cells.P);
  return hipGetLastError();
}

hipError_t launch_cell_params_on(rt_ctx c, int64_t n, const double* T, const double* x,
                                 const double* p, const CellSet& cells, hipStream_t s) {
  const int threads = 256;
  const int64_t blocks = (n + threads - 1) / threads;
  hipLaunchKernelGGL(cell_params_kernel, dim3((unsigned)blocks), dim3(threads), 0, s, n, T, x, p,
                     c->T_ref, c->dnu, second_radiation_cm_K(), c->have_E ? 1 : 0, cells.G,
                     cells.beta, cells.theta, cells.lam2, cells.P);
  return hipGetLastError();
}

hipError_t launch_cell_params32(rt_ctx c) {
  const int64_t n = c->n_cells;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(cell_params32_kernel, dim3(blocks), dim3(256), 0, c->stream, n, c->cells.uf,
                     c->cells.lamf, c->have_E ? 1 : 0, c->cells.Gq);
  for (int g = 1; g < kMaxGases; ++g) {
    const ExtraGas& gs = c->gas[g - 1];
    if (!gs.active) continue;
    hipLaunchKernelGGL(cell_params32_kernel, dim3(blocks), dim3(256), 0, c->stream, n, gs.uf,
                       c->cells.lamf, gs.have_E ? 1 : 0, gs.Gq);
  }
  return hipGetLastError();
}

hipError_t launch_gas_factor(rt_ctx c, int g) {
  const ExtraGas& gs = c->gas[g - 1];
  const int64_t n = c->n_cells;
  hipLaunchKernelGGL(gas_factor_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream,
                     n, c->d_T, gs.x, c->d_p, c->T_ref, c->dnu, gs.have_E ? 1 : 0, gs.G);
  return hipGetLastError();
}

// One form of the line sum: a.n_tiles tiles (of the form's points) and a.parts
// shares for `groups` groups of cells, and `walls` blocks of the walls' row.
template <int FORM, int P>
static hipError_t launch_sum(KappaArgs a, int64_t groups, int64_t walls, hipStream_t s) {
  constexpr int threads = FORM == kPrecSum ? kPrecThreads : kKappaThreads;
  hipError_t e = hipSuccess;
  const bool fits = for_pieces(
      groups, (int64_t)a.n_tiles * a.parts, walls, threads,
      [&](int64_t first, int64_t, int64_t blocks, bool last) {
        a.group0 = first;
        a.wall.first = last && walls ? (unsigned)blocks : 0xffffffffu;
        hipLaunchKernelGGL((kappa_linesum_kernel<FORM, P>),
                           dim3((unsigned)(blocks + (last ? walls : 0))), dim3(threads), 0, s, a);
        e = hipGetLastError();
        return e == hipSuccess;
      });
  return fits || e != hipSuccess ? e : hipErrorInvalidValue;
}

// The plain line sum of a.n_tiles tiles of kKappaTilePoints points for
// `groups` groups of cells, or of twice as many tiles of half the points, with
// the same values bit for bit (of whole sums: a tile's shares, a.parts > 1, are cut
// from the lines that meet the tile).  Half tiles have six wavefronts a SIMD instead
// of five and a tail half as long, and form a line's parameters and a span's
// interpolation from its far nodes in more blocks.  They win (whole against
// half tiles, microseconds):
// - in launches of few blocks, below 6 a CU: 1,344 blocks, windows of +-500
//   points, 0.25 lines a point 114, 105 (and 1,932 blocks 141, 141; 6,912 391,
//   448);
// - where windows of up to +-256 points leave the far nodes little: +-100
//   points, 0.5 and 6.5 lines a point, 19,200 blocks 1112, 1040 and 19,621,
//   16,190, 1,539 blocks 162, 117 and 2512, 1687; +-250, 1.2 lines, 19,200
//   blocks 4091, 3660;
// - where the list is dense enough that its lines outweigh a span's fixed
//   work, unless the window makes the parameters of the lines around a tile the
//   larger part: +-500, 1 line a point, 19,200 blocks 4535, 4440, 1,539 blocks
//   543, 460 (0.25 a point, 19,200 blocks: 924, 1062); +-1000, 1 line a point
//   3672, 4155.
// With a walls' row (a.wall.out) its blocks follow.  Tables of more blocks than a
// launch holds (137 GB in half tiles) take several.
static hipError_t launch_plain(rt_ctx c, KappaArgs a, int64_t groups, hipStream_t s) {
  const int64_t blocks = groups * a.n_tiles * a.parts;
  const int64_t walls = a.wall.out ? a.wall.ld / kKappaThreads : 0;
  const double lines_per_point = (double)a.t.L.n / ((double)a.t.n_nu + 2.0 * a.t.K);
  if (blocks < 6 * c->cus || a.t.K <= 256 || (a.t.K <= 512 && lines_per_point >= 0.9)) {
    a.n_tiles *= 2;
    a.tile_begin *= 2;
    return launch_sum<kPlainSum, 1>(a, groups, walls, s);
  }
  return launch_sum<kPlainSum, kKappaPoints>(a, groups, walls, s);
}

hipError_t launch_kappa(rt_ctx c, bool compensated) {
  KappaArgs a;
  if (!compensated && !c->planck) a.wall = wall_row_of(c);
  a.t.L = c->lines;
  a.t.C = c->cells;
  a.t.n_cells = c->n_cells;
  a.t.n_nu = c->n_nu;
  a.t.K = c->K;
  a.t.have_E = c->have_E ? 1 : 0;
  a.t.out = c->kappa;
  a.t.ld_out = c->ld;
  a.t.col0 = 0;
  a.t.col_end = c->ld;
  a.n_tiles = (int)((c->ld + kKappaTilePoints - 1) / kKappaTilePoints);
  a.tile_begin = 0;
  const int64_t groups = (c->n_cells + kKappaCells - 1) / kKappaCells;
  auto launch = [&]() {
    if (!compensated) return launch_plain(c, a, groups, c->stream);
    // the precision form: FP32 line parameters
    return launch_sum<kPrecSum, kKappaPoints>(a, groups, 0, c->stream);
  };
  hipError_t e = launch();
  a.wall.out = nullptr;  // written
  // further gases add their line sums, each with its own lines and G
  for (int g = 1; g < kMaxGases && e == hipSuccess; ++g) {
    const ExtraGas& gs = c->gas[g - 1];
    if (!gs.active) continue;
    a.t.L = gs.lines;
    a.t.C.G = gs.G;
    a.t.C.Gq = gs.Gq;
    a.t.have_E = gs.have_E ? 1 : 0;
    a.t.accumulate = 1;
    e = launch();
  }
  return e;
}

hipError_t launch_kappa_tiles(rt_ctx c, const KappaTile& t, int64_t n_cell_groups,
                              int tile_begin, int n_tiles, bool comp, hipStream_t s,
                              const TileGate& gate, int parts, int64_t part_stride) {
  KappaArgs a;
  a.t = t;
  a.gate = gate;
  a.n_tiles = n_tiles;
  a.tile_begin = tile_begin;
  a.parts = parts < 1 ? 1 : parts;
  a.part_stride = part_stride;
  if (!comp) return launch_plain(c, a, n_cell_groups, s);
  // the compensated sum has its own tiles of 256 points
  a.n_tiles *= kKappaPoints;
  a.tile_begin *= kKappaPoints;
  return launch_sum<kCompSum, 1>(a, n_cell_groups, 0, s);
}

// The plain line sum in 256-point tiles (one span per wavefront): twice the
// blocks of launch_kappa_tiles, each with half its work, for launches that
// cover only part of the table (the learned form's fallback), where the
// latency of one block rather than the total work sets the time.  The
// values are the same bit for bit.
hipError_t launch_kappa_tiles_fine(rt_ctx c, const KappaTile& t, int64_t n_cell_groups,
                                   int n_tiles, hipStream_t s, const TileGate& gate) {
  KappaArgs a;
  a.t = t;
  a.gate = gate;
  a.n_tiles = n_tiles;
  a.tile_begin = 0;
  return launch_sum<kPlainSum, 1>(a, n_cell_groups, 0, s);
}

hipError_t launch_planck_cubics(rt_ctx c, const double* theta, int64_t n, float4* poly,
                                hipStream_t s) {
  const int64_t chunks = plain_chunks(c->n_nu), blocks = (n * chunks + 255) / 256;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(planck_cubics_kernel, dim3((unsigned)blocks), dim3(256), 0, s, theta, n,
                     chunks, c->nu0, c->dnu, first_radiation_wavenumber(), poly);
  return hipGetLastError();
}

hipError_t launch_planck(rt_ctx c) {
  const dev::WallRow wall = wall_row_of(c);
  const int tiles = (int)(c->ld / 256);
  const int64_t n = c->planck ? c->n_cells : 0;
  const int64_t blocks = ((n + kPlanckCells - 1) / kPlanckCells + 1) * tiles;
  const unsigned gx = (unsigned)std::min<int64_t>(blocks, 65536);
  const unsigned gy = (unsigned)((blocks + gx - 1) / gx);
  hipLaunchKernelGGL(planck_table_kernel, dim3(gx, gy), dim3(256), 0, c->stream, c->cells.theta2,
                     n, c->n_nu, c->ld, tiles, wall.nu0, wall.dnu, wall.c1, c->planck, wall);
  return hipGetLastError();
}

}  // namespace rt
