// march.hip -- Monte-Carlo rays through the cell grid on gfx950.
//
//   order      : a coherent processing order for the rays of a batch
//                (counting sort on a direction/position key)
//   raygen_dda : Philox4x64-10 ray sampling (uniform boundary point,
//                cosine-weighted inward direction) and exact integer
//                traversal -> per-ray list of (cell, length) segments
//   march      : Eq. (3) applied cell after cell for every nu point; each
//                wavefront owns one ray and one spectral chunk
//                (dev::march_plain, dev::march_prec); the absorbed and emitted power of the
//                chunk per segment is summed across the wavefront in a fixed
//                order and added to the cell's fixed-point accumulator
//   tally      : the accumulators as FP64 powers per cell, and the energy
//                balance from exact sums of the accumulators
#include "device_common.h"

#include <cmath>

namespace rt {
namespace {

using namespace dev;

__global__ void order_key_kernel(uint64_t seed, uint64_t begin, int64_t count, int nx, int ny,
                                 int nz, uint32_t* keys, uint32_t* hist) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  int64_t O[3], D[3];
  sample_ray(seed, begin + (uint64_t)i, nx, ny, nz, O, D);
  const uint32_t k = order_key(O, D, nx, ny, nz);
  keys[i] = k;
  atomicAdd(hist + k, 1u);
}

__global__ void order_scatter_kernel(const uint32_t* __restrict__ keys, int64_t count,
                                     uint32_t* offsets, uint32_t* perm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  perm[atomicAdd(offsets + keys[i], 1u)] = (uint32_t)i;
}

__global__ void zero_u32_kernel(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// Slot i of the batch holds ray begin + perm[i] (begin + i without perm).
__global__ void raygen_dda_kernel(uint64_t seed, uint64_t begin, int64_t count, int nx, int ny,
                                  int nz, double unit_cm, int max_segs,
                                  const int64_t* __restrict__ explicit_rays, int64_t* rays_out,
                                  int2* segs, int32_t* counts, unsigned long long* seg_total,
                                  const uint32_t* __restrict__ perm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int ns = 0;
  if (i < count) {
    int64_t O[3], D[3];
    if (explicit_rays) {
      for (int k = 0; k < 3; ++k) {
        O[k] = explicit_rays[6 * i + k];
        D[k] = explicit_rays[6 * i + 3 + k];
      }
    } else {
      sample_ray(seed, begin + (perm ? (uint64_t)perm[i] : (uint64_t)i), nx, ny, nz, O, D);
    }
    if (rays_out)
      for (int k = 0; k < 3; ++k) {
        rays_out[6 * i + k] = O[k];
        rays_out[6 * i + 3 + k] = D[k];
      }
    ns = traverse(nx, ny, nz, unit_cm, O, D, max_segs, segs + i * max_segs);
    counts[i] = ns;
  }
  // one atomic per wavefront for the work counter
  unsigned long long v = (unsigned long long)ns;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if (seg_total && (threadIdx.x & 63) == 0 && v) atomicAdd(seg_total, v);
}

struct MarchArgs {
  MarchWave w;
  int64_t ray_blocks_x;  // ray blocks per XCD
  const int2* segs;
  const int32_t* counts;
  int max_segs;
  int64_t n_rays;
  float* exit_I;
};

// Block = 4 wavefronts = 4 consecutive rays (batch slots) on one spectral
// chunk (blockIdx.y).  Workgroups are dispatched to the 8 XCDs round-robin, so
// block b of a chunk runs on XCD b % 8 (a chunk's blocks are a multiple of 8);
// that XCD is given a contiguous range of ray blocks, chunk-major, so the
// waves in flight on it march neighbouring rays of the coherent order through
// one chunk and share kappa rows in its L2.
__device__ __forceinline__ bool march_place(const MarchArgs& a, int64_t& ray, int& wave,
                                            int& lane) {
  const unsigned b = blockIdx.x;
  const int64_t rb = (int64_t)(b & 7) * a.ray_blocks_x + (b >> 3);
  wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  lane = threadIdx.x & 63;
  ray = rb * 4 + wave;
  return ray < a.n_rays;
}

// Plain form (see march_plain).
template <bool EXIT, bool CUBIC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8))) void march_kernel(
    MarchArgs a) {
  __shared__ float stage[4][PlainStage::kEntries];
  int64_t ray;
  int wave, lane;
  if (!march_place(a, ray, wave, lane)) return;
  march_plain<EXIT, CUBIC, true>(a.w, a.segs + ray * a.max_segs, a.counts[ray],
                                 (int64_t)blockIdx.y * kMarchPoints, lane,
                                 EXIT ? a.exit_I + ray * a.w.ld : nullptr, stage[wave], ray);
}

// Precision form (Planck table, FP64 partial sums).
template <bool EXIT, int Q>
__global__ __launch_bounds__(256) void march_prec_kernel(MarchArgs a) {
  __shared__ double stage[4][PrecStage::kEntries];
  int64_t ray;
  int wave, lane;
  if (!march_place(a, ray, wave, lane)) return;
  march_prec<EXIT, Q>(a.w, a.segs + ray * a.max_segs, a.counts[ray], (int64_t)blockIdx.y * 64 * Q,
                      lane, EXIT ? a.exit_I + ray * a.w.ld : nullptr, stage[wave], ray);
}

// Carries of every accumulator row (rows x 2 digit groups).
__global__ void acc_normalize_kernel(unsigned long long* acc, int64_t groups) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < groups) acc_normalize(acc + i * kAccDigits);
}

// Digit sums of a block's 256 rows in thread 0: in the wavefront by lane
// exchanges, then over the four wavefronts.
__device__ void acc_block_sum(unsigned long long (&d)[kAccRow]) {
  __shared__ unsigned long long red[3][kAccRow];
#pragma unroll
  for (int k = 0; k < kAccRow; ++k)
    for (int off = 32; off > 0; off >>= 1) d[k] += __shfl_xor(d[k], off);
  const int wave = threadIdx.x >> 6;
  __syncthreads();  // an earlier sum's rows read
  if (wave > 0 && (threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < kAccRow; ++k) red[wave - 1][k] = d[k];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < kAccRow; ++k) d[k] += red[0][k] + red[1][k] + red[2][k];
}

// Per-cell powers from the normalised accumulators, and balance = {entering,
// sum emitted, sum absorbed, escaped}, each from the exact sum of its
// accumulators (cells, or the balance rows), converted once.  A block adds its
// cells' digits to the handle's sums (normalised digits are below 2^28 and
// there are fewer than 2^31 cells), the last block of the grid those of the
// balance rows; the last block to finish converts the sums and leaves them and
// the ticket cleared.  out: absorbed[n], emitted[n], balance[4], overflow flag.
// sums: cells' digits, balance digits, ticket.
//
// A chain of loads, exchanges and atomics: 8 us at 512 cells (a launch over
// the cells and one of a single block over all rows took 4 and 11 with a gap of
// 5), and 53 against 133 a call with its copies at 32^3 cells.
__global__ __launch_bounds__(256) void tally_kernel(const unsigned long long* __restrict__ acc,
                                                    int64_t n_cells, int copies, int64_t rows,
                                                    unsigned long long* sums, double* out) {
  __shared__ bool last;
  const bool bal = blockIdx.x == gridDim.x - 1;
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  unsigned long long d[kAccRow];
  if (bal) {
    acc_sum_copies(acc + rows * kAccRow, threadIdx.x, 256, kBalRows / 256, d);
  } else if (c < n_cells) {
    acc_sum_copies(acc, c, n_cells, copies, d);
    out[c] = acc_value(d);
    out[n_cells + c] = acc_value(d + kAccDigits);
  } else {
#pragma unroll
    for (int k = 0; k < kAccRow; ++k) d[k] = 0;
  }
  acc_block_sum(d);
  unsigned long long* const ticket = sums + 2 * kAccRow;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kAccRow; ++k) atomicAdd(sums + (bal ? kAccRow : 0) + k, d[k]);
    __threadfence();
    last = atomicAdd(ticket, 1ull) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last || threadIdx.x > 4) return;
  double* const balance = out + 2 * n_cells;
  if (threadIdx.x == 4) {  // the flag behind the balance rows
    balance[4] = *reinterpret_cast<const unsigned*>(acc + (rows + kBalRows) * kAccRow) ? 1.0 : 0.0;
    atomicExch(ticket, 0ull);
    return;
  }
  // absorbed, emitted, entering, escaped
  unsigned long long v[kAccDigits];
#pragma unroll
  for (int k = 0; k < kAccDigits; ++k) v[k] = atomicExch(sums + threadIdx.x * kAccDigits + k, 0ull);
  acc_normalize(v);
  const int at[4] = {2, 1, 0, 3};
  balance[at[threadIdx.x]] = acc_value(v);
}

// Clears the accumulators (and the overflow flag behind them), the segment
// count and, where given, the kept evaluations.
__global__ void zero_tally_kernel(unsigned long long* acc, int64_t n, unsigned long long* segs,
                                  unsigned long long* evals) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) acc[i] = 0;
  if (i == 0) {
    *segs = 0;
    if (evals) *evals = 0;
  }
}

// Exclusive prefix sums of n histograms in place.  A histogram is
// kOrderTiles tiles of 1024 buckets: first the tiles' sums, then every tile's
// block adds the sums before its own.  Both are launches of a few
// microseconds (4.3 and 4.4 us; one block per histogram, each thread over a
// run of 216 buckets at a stride that no two lanes share a line of, took 360).
__global__ __launch_bounds__(256) void order_sums_kernel(const uint32_t* __restrict__ hist,
                                                         uint32_t* sums) {
  __shared__ uint32_t part[4];
  const int64_t h = blockIdx.y;
  const uint4 v =
      reinterpret_cast<const uint4*>(hist + h * kOrderBuckets)[blockIdx.x * 256 + threadIdx.x];
  uint32_t s = v.x + v.y + v.z + v.w;
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) sums[h * kOrderTiles + blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

__global__ __launch_bounds__(256) void order_scan_kernel(uint32_t* hist,
                                                         const uint32_t* __restrict__ sums) {
  __shared__ uint32_t part[8];
  const int64_t h = blockIdx.y;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // the tiles before this one (kOrderTiles <= 256: one per thread)
  uint32_t before = t < (int)blockIdx.x ? sums[h * kOrderTiles + t] : 0u;
  for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
  uint4* p = reinterpret_cast<uint4*>(hist + h * kOrderBuckets) + blockIdx.x * 256 + t;
  const uint4 v = *p;
  const uint32_t own = v.x + v.y + v.z + v.w;
  uint32_t incl = own;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(incl, off);
    if (lane >= off) incl += u;
  }
  if (lane == 0) part[wave] = before;
  if (lane == 63) part[4 + wave] = incl;
  __syncthreads();
  uint32_t base = part[0] + part[1] + part[2] + part[3] + incl - own;
  for (int w = 0; w < wave; ++w) base += part[4 + w];
  *p = make_uint4(base, base + v.x, base + v.x + v.y, base + v.x + v.y + v.z);
}

}  // namespace

hipError_t launch_order_scan(uint32_t* hist, uint32_t* sums, int n, hipStream_t s) {
  for (int h = 0; h < n; h += 32768) {  // a grid's y ends at 65,535
    const dim3 grid(kOrderTiles, (unsigned)std::min(n - h, 32768));
    uint32_t* const hh = hist + (int64_t)h * kOrderBuckets;
    uint32_t* const hs = sums + (int64_t)h * kOrderTiles;
    hipLaunchKernelGGL(order_sums_kernel, grid, dim3(256), 0, s, hh, hs);
    hipLaunchKernelGGL(order_scan_kernel, grid, dim3(256), 0, s, hh, hs);
  }
  return hipGetLastError();
}

RayScratch owned_rays(rt_ctx c) {
  RayScratch s;
  s.segs = c->d_segs;
  s.counts = c->d_counts;
  s.keys = c->d_keys;
  s.perm = c->d_perm;
  s.hist = c->d_hist;
  s.max_segs = c->max_segs;
  s.cap = c->batch_rays;
  return s;
}

hipError_t launch_order(rt_ctx c, const RayScratch& s, uint64_t seed, uint64_t begin,
                        int64_t count) {
  const int threads = 256;
  const unsigned blocks = (unsigned)((count + threads - 1) / threads);
  hipLaunchKernelGGL(zero_u32_kernel, dim3((kOrderBuckets + threads - 1) / threads), dim3(threads),
                     0, c->stream, s.hist, (int64_t)kOrderBuckets);
  hipLaunchKernelGGL(order_key_kernel, dim3(blocks), dim3(threads), 0, c->stream, seed, begin,
                     count, c->nx, c->ny, c->nz, s.keys, s.hist);
  hipError_t e = launch_order_scan(s.hist, s.perm, 1, c->stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(order_scatter_kernel, dim3(blocks), dim3(threads), 0, c->stream, s.keys,
                     count, s.hist, s.perm);
  return hipGetLastError();
}

hipError_t launch_raygen(rt_ctx c, const RayScratch& s, uint64_t seed, uint64_t begin,
                         int64_t count, bool explicit_rays, int64_t* rays_out, bool count_work,
                         const uint32_t* perm) {
  const int threads = 256;
  const int64_t blocks = (count + threads - 1) / threads;
  const double unit_cm = c->cell_m * 100.0 / (double)kCellUnits;
  hipLaunchKernelGGL(raygen_dda_kernel, dim3((unsigned)blocks), dim3(threads), 0, c->stream,
                     seed, begin, count, c->nx, c->ny, c->nz, unit_cm, s.max_segs,
                     explicit_rays ? c->d_rays_explicit : nullptr, rays_out, s.segs,
                     s.counts, count_work ? c->d_segcount : nullptr, perm);
  return hipGetLastError();
}

int64_t plain_chunks(int64_t n_nu) { return (n_nu + kMarchPoints - 1) / kMarchPoints; }

// The Planck cubics serve a grid where, over its temperatures and wavenumbers
// (checked at the extremes and midpoints of both ranges), a chunk's cubic is
// within 2^-25 of B and the first-order expansion over a lane's kPlainQ points
// within 2^-24 (FP32 unit roundoff) of it: at 300 K and 1000 cm^-1 up to
// dnu of about 0.03 cm^-1.  A cubic costs the march 7 instructions per
// segment against 17 for the general value, and 16 bytes per row of 3 KB.
bool planck_cubic_fits(double T_min, double T_max, double nu0, double dnu, int n_nu) {
  const double c2 = second_radiation_cm_K();
  const double half = 0.5 * kMarchPoints;
  auto B = [&](double nu, double T) { return nu * nu * nu / std::expm1(c2 * nu / T); };
  const double mid0 = nu0 + 0.5 * (kMarchPoints - 1) * dnu;
  const double last = (double)(plain_chunks(n_nu) - 1) * kMarchPoints * dnu;
  const double u[5] = {-1.0, -0.7071, 0.0, 0.7071, 1.0};
  for (double T : {T_min, T_max, std::sqrt(T_min * T_max)})
    for (double m : {mid0, mid0 + 0.5 * last, mid0 + last}) {
      const double x[4] = {-kCubicNodeA, -kCubicNodeB, kCubicNodeB, kCubicNodeA};
      double f[4], r[4];
      for (int i = 0; i < 4; ++i) f[i] = B(m + x[i] * half * dnu, T);
      planck_cubic(f, half, r);
      for (double v : u) {
        const double p = v * half, ref = B(m + p * dnu, T);
        const double fit = r[0] + p * (r[1] + p * (r[2] + p * r[3]));
        if (!(std::fabs(fit - ref) <= std::ldexp(ref, -25))) return false;
        const double d2 = 0.5 * std::fabs(2.0 * r[2] + 6.0 * r[3] * p) * (kPlainQ - 1) * (kPlainQ - 1);
        if (!(d2 < std::ldexp(ref, -24))) return false;
      }
    }
  return true;
}

// Where the visits of a cell's rows (of n_rays_total rays, a mean path of 3 /
// (1/nx + 1/ny + 1/nz) segments) are few for the size of the grid, the rows
// come from beyond L2 and 4 points per lane are faster.  The line, at 20,000
// points (8 against 4, microseconds; 6,000 and 10,000 points cross at the same
// visits): 14^3 cells, 40 visits 1988, 1810; 80 3064, 3374.  16^3, 80 5142, 5026;
// 120 7182, 7446.  18^3, 120 11,634, 10,761; 160 13,835, 14,282.  20^3, 160 20,862,
// 19,741; at 10,000 points 200 visits 11,790, 12,543.  24^3, 10,000 points, 200
// 22,735, 21,596; 6,000 points, 250 15,847, 16,244.  12^3, 40 1082, 1108.  It
// depends on the ray set and not on the part of it in a call, so that every split
// of a set adds the same sums.
int prec_points(rt_ctx c, double n_rays_total) {
  const double cells = (double)c->n_cells;
  const double segs = 3.0 / (1.0 / c->nx + 1.0 / c->ny + 1.0 / c->nz);
  return cells >= 2048 && n_rays_total * segs / cells <= std::min(cells / 50, 200.0) &&
                 c->n_nu <= (1 << 22)  // a grid's y ends at 65,535
             ? 4
             : 8;
}

// prec_q: points per lane of the precision form, 0 for the plain form.
int64_t march_chunks(int64_t n_nu, int prec_q) {
  return prec_q ? (n_nu + 64 * prec_q - 1) / (64 * prec_q) : plain_chunks(n_nu);
}

hipError_t launch_march(rt_ctx c, const RayScratch& s, int64_t count, double weight, int prec_q,
                        float* exit_dev) {
  MarchArgs a;
  a.w.kappa = c->kappa;
  a.w.planck = c->planck;
  a.w.ld = c->ld;
  a.w.col0 = 0;
  a.w.theta = c->cells.theta;
  a.w.poly = c->d_poly;
  a.w.n_poly = plain_chunks(c->n_nu);
  a.w.bwall = c->d_bwall;
  a.w.nu0 = c->nu0;
  a.w.dnu = c->dnu;
  a.w.c1 = first_radiation_wavenumber();
  a.w.weight = weight;
  a.w.acc = c->d_acc;
  a.w.row0 = 0;
  a.w.rep_rows = c->n_cells;
  a.w.rep_mask = acc_copies(c->n_cells) - 1;
  a.w.bal_row0 = c->acc_rows;
  a.w.bal_mask = kBalRows - 1;
  a.w.ovf = c->d_ovf;
  a.ray_blocks_x = ((count + 3) / 4 + 7) / 8;
  a.segs = s.segs;
  a.counts = s.counts;
  a.max_segs = s.max_segs;
  a.n_rays = count;
  a.exit_I = exit_dev;
  // the columns past n_nu hold zeros and add nothing: the march stops at the
  // last chunk that holds a point
  const int64_t n_chunks = march_chunks(c->n_nu, prec_q);
  // x: at most 2^21 rays a batch, 2^19 blocks; y: n_nu < 2^24 points, 2^15 chunks
  const dim3 g((unsigned)(8 * a.ray_blocks_x), (unsigned)n_chunks), t(256);
  // Plain form: seven wavefronts per SIMD.  32^3 cells, 50,000 points, eight, seven
  // and six: 2^18 rays 168, 155, 145 ms, 2^20 500, 502, 510; 24^3, 20,000 points,
  // 32,768 rays 8.23, 7.94, 7.63
  const unsigned pad = 6000;
  if (prec_q == 4) {
    if (exit_dev) hipLaunchKernelGGL((march_prec_kernel<true, 4>), g, t, 0, c->stream, a);
    else hipLaunchKernelGGL((march_prec_kernel<false, 4>), g, t, 0, c->stream, a);
  } else if (prec_q) {
    if (exit_dev) hipLaunchKernelGGL((march_prec_kernel<true, 8>), g, t, 0, c->stream, a);
    else hipLaunchKernelGGL((march_prec_kernel<false, 8>), g, t, 0, c->stream, a);
  } else if (c->planck_cubic) {
    if (exit_dev) hipLaunchKernelGGL((march_kernel<true, true>), g, t, pad, c->stream, a);
    else hipLaunchKernelGGL((march_kernel<false, true>), g, t, pad, c->stream, a);
  } else {
    if (exit_dev) hipLaunchKernelGGL((march_kernel<true, false>), g, t, pad, c->stream, a);
    else hipLaunchKernelGGL((march_kernel<false, false>), g, t, pad, c->stream, a);
  }
  const int64_t groups = 2 * (c->acc_rows + kBalRows);
  hipLaunchKernelGGL(acc_normalize_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0,
                     c->stream, c->d_acc, groups);
  return hipGetLastError();
}

hipError_t launch_tally(rt_ctx c, double* out) {
  hipLaunchKernelGGL(tally_kernel, dim3((unsigned)((c->n_cells + 255) / 256 + 1)), dim3(256), 0,
                     c->stream, c->d_acc, c->n_cells, acc_copies(c->n_cells), c->acc_rows,
                     c->d_tally_sums, out);
  return hipGetLastError();
}

hipError_t launch_zero(rt_ctx c, bool evals) {
  const int64_t n = (c->acc_rows + kBalRows) * kAccRow + 1;
  hipLaunchKernelGGL(zero_tally_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream,
                     c->d_acc, n, c->d_segcount, evals ? c->d_adapt_evals : nullptr);
  return hipGetLastError();
}

}  // namespace rt
