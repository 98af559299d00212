// kde_kernels.hip -- gfx950 kernels for exact bandwidth-selection pair sums.
//
// Method: Andrzejewski, Gramacki, Gramacki, arXiv 1505.01998, Section 4.4
// (selectors), Section 4.5 (pair distance reused across bandwidths) and
// Section 5.4 (sums of a function of X_i - X_j over the i < j triangle).
//
// Jobs.  Every call works on a set of columns (one for the single-column
// selectors, many for a batch).  Column descriptors (ColDesc) say where each
// column's samples, grid coefficients and partial sums live; every pair
// kernel block decodes one work unit (Unit: column, row of samples i, j-range,
// bandwidth chunk), so units of different columns share a launch.
//
// Pair kernels.  A block of 256 threads (four 64-wide waves) owns a "row" of
// 256 consecutive samples i, one per lane, held in a register for the whole
// block.  The block sweeps a j-range of the triangle in tiles of kBJ samples
// that are staged in LDS with coalesced 16-byte loads; every lane of a wave
// reads the same LDS address (a broadcast), so each wave walks j in lockstep
// against its 64 register-resident i.  Because j is wave-uniform, loop bounds
// are uniform and nothing diverges; the only masking is the 64x64 diagonal
// block of each wave, where pairs with j <= i are given an infinite squared
// distance (exp2(-inf) = 0 exactly).  Padded samples beyond n hold +inf and
// contribute exactly zero the same way; padded lanes (i >= n) are dropped
// when the block's partial sums are formed.
//
// Precision (mixed form).  Pair terms are FP32 (v_exp_f32).  Each lane sums
// 64 consecutive j in plain FP32, then folds that run into an FP64
// accumulator (the LSCV sweep: a conversion and an FP64 add, which issue at
// the unpacked FP32 rate, half the cost of a compensated FP32 fold) or a
// Kahan-compensated FP32 one (the psi pass, two sums per 64 pairs).  Lane
// accumulators are reduced in FP64 across the wave (lane exchanges), the
// block (LDS, fixed order) and the work items (a separate row-reduction
// kernel, fixed order), so the result is deterministic and independent of
// scheduling.  The FP64 form
// computes every term and sum in FP64.
#include <hip/hip_runtime.h>
#include <math.h>

#include "kde_internal.h"

namespace kde {

namespace {

constexpr float kInfF = __builtin_inff();
constexpr double kInfD = __builtin_inf();
constexpr double kPi = 3.14159265358979323846;
constexpr double kLog2E = 1.4426950408889634074;
constexpr int kRun = 64;  // j per plain-FP32 run before a compensated fold
// Squared scaled distance beyond which a psi term is zero in FP32; clamping
// keeps the Hermite polynomial finite when the distance is huge or infinite.
constexpr float kWMax = 4096.0f;
// A column whose scaled copy (samples / g) spans at most this range has every
// squared scaled distance below 4e8, where He_8 stays far inside the FP32
// range, so its psi sweep needs no clamp except on masked and padded pairs.
constexpr double kPsiFastRange = 2.0e4;
// exp2 factor of the psi term: e^(-w/2) = exp2(w * kPsiExp2)
constexpr float kPsiExp2 = (float)(-0.5 * 1.4426950408889634074);

__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] += sh[t + s];
    __syncthreads();
  }
  double r = sh[0];
  __syncthreads();
  return r;
}

// Block-wide minimum and maximum (every thread receives both).
__device__ __forceinline__ void block_minmax(float& lo, float& hi, float* sh) {
  const int t = threadIdx.x;
  sh[t] = lo;
  sh[kThreads + t] = hi;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if (t < s) {
      sh[t] = fminf(sh[t], sh[t + s]);
      sh[kThreads + t] = fmaxf(sh[kThreads + t], sh[kThreads + t + s]);
    }
    __syncthreads();
  }
  lo = sh[0];
  hi = sh[kThreads];
  __syncthreads();
}

// A wave-uniform float kept in a scalar register: the bandwidth coefficients
// of the LSCV sweeps are the same for every lane, and holding them in SGPRs
// instead of VGPRs frees HC vector registers per lane (more waves per SIMD).
__device__ __forceinline__ float uniform_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Kahan fold of a run sum r into (acc, comp); the compensated value is acc - comp.
__device__ __forceinline__ void kahan_add(float& acc, float& comp, float r) {
  const float y = r - comp;
  const float t = acc + y;
  comp = (t - acc) - y;
  acc = t;
}

// Probabilists' Hermite polynomial He_r(u) as a polynomial in w = u^2.
template <int R>
__device__ __forceinline__ float herm_w(float w);
template <>
__device__ __forceinline__ float herm_w<4>(float w) {
  return __builtin_fmaf(w - 6.0f, w, 3.0f);
}
template <>
__device__ __forceinline__ float herm_w<6>(float w) {
  float p = __builtin_fmaf(w - 15.0f, w, 45.0f);
  return __builtin_fmaf(p, w, -15.0f);
}
template <>
__device__ __forceinline__ float herm_w<8>(float w) {
  float p = __builtin_fmaf(w - 28.0f, w, 210.0f);
  p = __builtin_fmaf(p, w, -420.0f);
  return __builtin_fmaf(p, w, 105.0f);
}
template <int R>
__device__ __forceinline__ double herm_w64(double w);
template <>
__device__ __forceinline__ double herm_w64<4>(double w) {
  return __builtin_fma(w - 6.0, w, 3.0);
}
template <>
__device__ __forceinline__ double herm_w64<6>(double w) {
  double p = __builtin_fma(w - 15.0, w, 45.0);
  return __builtin_fma(p, w, -15.0);
}
template <>
__device__ __forceinline__ double herm_w64<8>(double w) {
  double p = __builtin_fma(w - 28.0, w, 210.0);
  p = __builtin_fma(p, w, -420.0);
  return __builtin_fma(p, w, 105.0);
}

// He_r(0) = (-1)^(r/2) (r-1)!! for even r, from the recurrence
// He_{k+1}(0) = -k He_{k-1}(0) with He_0(0) = 1: the kernel-derivative value
// K^(r)(0) = He_r(0) / sqrt(2 pi) (r = 4, 6, 8) and the normal-scale
// functionals below (r = 8, 10).
__device__ __forceinline__ double herm_at0(int r) {
  double h = 1.0;
  for (int k = 1; k < r; k += 2) h *= -(double)k;
  return h;
}

// Normal-scale functional psi_r of N(0, sigma^2): the integral of f^(r) f
// for the normal density is He_r(0) / (2^(r/2+1) sqrt(pi) sigma^(r+1)) (the
// convolution of two N(0, sigma^2) densities is N(0, 2 sigma^2), whose r-th
// derivative at 0 is He_r(0) / (sqrt(2 pi) (sqrt(2) sigma)^(r+1))); r = 8
// gives the printed 105 / (32 sqrt(pi) sigma^9).
__device__ double psi_normal_scale(int r, double sigma) {
  return herm_at0(r) / (ldexp(1.0, r / 2 + 1) * sqrt(kPi) * pow(sigma, (double)(r + 1)));
}

// ------------------------------------------------------------------ statistics
__device__ __forceinline__ double load_raw(const ColDesc& c, int i) {
  return c.raw_f64 ? reinterpret_cast<const double*>(c.raw)[i] : (double)reinterpret_cast<const float*>(c.raw)[i];
}

__device__ __forceinline__ int stat_blocks(int n) { return min(kStatBlocks, (n + 2047) / 2048); }

// Pass 1: per-block FP64 sum of the samples and count of non-finite values;
// block blk of the column's stat_blocks.
__device__ void stats_sum(const ColDesc& c, int blk) {
  const int nblk = stat_blocks(c.n);
  if (blk >= nblk) return;
  __shared__ double sh[kThreads];
  __shared__ int nf_sh;
  const int chunk = (c.n + nblk - 1) / nblk;
  const int b0 = blk * chunk;
  const int b1 = min(c.n, b0 + chunk);
  if (threadIdx.x == 0) nf_sh = 0;
  __syncthreads();
  double s = 0.0;
  int nf = 0;
  for (int i = b0 + threadIdx.x; i < b1; i += kThreads) {
    const double v = load_raw(c, i);
    if (!isfinite(v)) ++nf; else s += v;
  }
  if (nf) atomicAdd(&nf_sh, nf);
  s = block_sum(s, sh);
  if (threadIdx.x == 0) {
    c.stat[blk] = s;
    c.stat_nf[blk] = nf_sh;
  }
}

// Mean of a column (by one block); float64 columns are shifted by it.
__device__ void stats_mean(const ColDesc& c) {
  const int nblk = stat_blocks(c.n);
  __shared__ double sh[kThreads];
  __shared__ int nf_sh;
  if (threadIdx.x == 0) nf_sh = 0;
  __syncthreads();
  double s = 0.0;
  int nf = 0;
  for (int b = threadIdx.x; b < nblk; b += kThreads) {
    s += c.stat[b];
    nf += c.stat_nf[b];
  }
  if (nf) atomicAdd(&nf_sh, nf);
  s = block_sum(s, sh);
  if (threadIdx.x == 0) {
    DevState& d = *c.st;
    d.n = (double)c.n;
    d.status = nf_sh ? kStInval : kStOk;
    d.mean = s / (double)c.n;
    d.shift = c.raw_f64 ? d.mean : 0.0;
  }
}

// Pass 2: per-block sum of squared deviations; writes the padded FP32 (and
// FP64) working copies of the column.
__device__ void stats_dev(const ColDesc& c, int blk) {
  const int nblk = stat_blocks(c.n);
  if (blk >= nblk) return;
  __shared__ double sh[kThreads];
  const double mean = c.st->mean, shift = c.st->shift;
  float* y32 = c.x32;
  double* y64 = c.x64;
  const int chunk = (c.n + nblk - 1) / nblk;
  const int b0 = blk * chunk;
  const int b1 = min(c.n, b0 + chunk);
  __shared__ float shm[2 * kThreads];
  double s = 0.0;
  float lo = kInfF, hi = -kInfF;
  for (int i = b0 + threadIdx.x; i < b1; i += kThreads) {
    const double v = load_raw(c, i);
    const double d = v - mean;
    s += d * d;
    const float w = (float)(v - shift);
    y32[i] = w;
    lo = fminf(lo, w);
    hi = fmaxf(hi, w);
    if (y64) y64[i] = v;
  }
  for (int i = c.n + blk * kThreads + threadIdx.x; i < c.n + kPad; i += nblk * kThreads) {
    y32[i] = kInfF;
    if (y64) y64[i] = kInfD;
  }
  s = block_sum(s, sh);
  block_minmax(lo, hi, shm);
  if (threadIdx.x == 0) {
    c.stat[blk] = s;
    c.stat_mm[blk] = lo;
    c.stat_mm[kStatBlocks + blk] = hi;
  }
}

// ------------------------------------------------------------------ plug-in scalar steps
// Each by one thread of a column.  Stage s in {0, 1, 2} estimates psi_r,
// r = 8 - 2 s.  A step that follows another one at once (the pass's lists name
// the same columns) runs at the end of that one's kernel: small calls are
// bound by the number of their launches, 2-4 us each.
__device__ void psi_begin(DevState& d, int stage) {
  d.active = 0;
  d.need_f64 = 0;
  if (d.status != kStOk || d.pstatus != kStOk || d.stages == 0) return;
  if (stage == 0 && d.stages != 3) return;
  const int r = 8 - 2 * stage;
  double psi_next;
  if (stage == 0) {
    psi_next = psi_normal_scale(10, d.sigma);
  } else if (stage == 1) {
    if (d.stages == 2) d.psi[0] = psi_normal_scale(8, d.sigma);
    psi_next = d.psi[0];
  } else {
    psi_next = d.psi[1];
  }
  // AMSE pilot: g = [-2 K^(r)(0) / (mu_2 psi_{r+2} n)]^(1/(r+3)), mu_2 = 1
  const double k0 = herm_at0(r) / sqrt(2.0 * kPi);
  const double rad = -2.0 * k0 / (psi_next * d.n);
  if (!(rad > 0.0) || !isfinite(rad)) {
    d.pstatus = kStDegenerate;
    return;
  }
  const double g = pow(rad, 1.0 / (double)(r + 3));
  d.active = 1;
  d.g[stage] = g;
  const double ig2 = 1.0 / (g * g);
  d.psi_scale = (float)(1.0 / g);
  d.psi_fast = ((double)d.xmax - (double)d.xmin) * (double)d.psi_scale <= kPsiFastRange ? 1 : 0;
  d.cd[0] = ig2;
  d.cd[1] = -0.5 * ig2;
}

__device__ void plugin_final(DevState& d) {
  if (d.status != kStOk || d.pstatus != kStOk || d.stages == 0) return;
  // h = [R(K) / (mu_2^2 psi_4 n)]^(1/5), R(K) = 1/(2 sqrt(pi))
  const double rad = (0.5 / sqrt(kPi)) / (d.psi[2] * d.n);
  if (!(rad > 0.0) || !isfinite(rad)) {
    d.pstatus = kStDegenerate;
    return;
  }
  d.h_plugin = pow(rad, 0.2);
}

__device__ __forceinline__ void plugin_step(DevState& d, int step) {
  if (step == kStepFinal)
    plugin_final(d);
  else if (step >= 0)
    psi_begin(d, step);
}

__global__ void k_plugin_step(const ColDesc* __restrict__ cols, const int* __restrict__ ids, int n_ids, int step) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_ids) plugin_step(*cols[ids[k]].st, step);
}

// Scaled copy of a large column for the mixed form's psi pass: y = x32 * (1/g)
// in FP32 (padding stays +inf).  Grid (blocks, columns); inactive columns are
// skipped.  Small columns are scaled as their units load them.
__global__ __launch_bounds__(kThreads) void k_psi_scale(const ColDesc* __restrict__ cols,
                                                        const int* __restrict__ ids) {
  const ColDesc c = cols[ids[blockIdx.y]];
  if (!c.st->active) return;
  const float s = c.st->psi_scale;
  const int m = c.n + kPad;
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < m; i += gridDim.x * kThreads)
    c.y32[i] = i < c.n ? c.x32[i] * s : kInfF;
}

// Block per column: psi_sums[0] = sum_{i<j} He_r(u) e^{-u^2/2}, psi_sums[1] =
// sum of its absolute value, u = (X_i - X_j)/g, from the units' partials in a
// fixed order, then psi_r = [2 sum K^(r) + n K^(r)(0)] / (n^2 g^(r+1)).
// conditional: this is the FP64 re-run of the mixed form; the stage stands
// unless flagged.  next: the step that follows (-1: none).
__global__ __launch_bounds__(kThreads) void k_psi_finish(const ColDesc* __restrict__ cols,
                                                         const int* __restrict__ ids, int stage, int was_f64,
                                                         int conditional, int next) {
  const ColDesc& c = cols[ids[blockIdx.x]];
  DevState& d = *c.st;
  __shared__ double sh[2][kThreads];
  const int t = threadIdx.x;
  const bool todo = d.active && !(conditional && !d.need_f64);  // uniform over the block
  __syncthreads();  // every wave has read the flags that thread 0 changes below
  if (todo) {
    const int m = c.n_items_psi;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 8
    for (int k = t; k < m; k += kThreads) {
      s0 += c.psi_part[k];
      s1 += c.psi_part[m + k];
    }
    sh[0][t] = s0;
    sh[1][t] = s1;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
      if (t < s) {
        sh[0][t] += sh[0][t + s];
        sh[1][t] += sh[1][t + s];
      }
      __syncthreads();
    }
  }
  if (t != 0) return;
  if (todo) {
    c.psi_sums[0] = sh[0][0];
    c.psi_sums[1] = sh[1][0];
    const int r = 8 - 2 * stage;
    const double inv_s2pi = 1.0 / sqrt(2.0 * kPi);
    const double n = d.n, g = d.g[stage];
    const double s = sh[0][0] * inv_s2pi, a = sh[1][0] * inv_s2pi;
    d.psi[stage] = (2.0 * s + n * herm_at0(r) * inv_s2pi) / (n * n * pow(g, (double)(r + 1)));
    d.kappa[stage] = (s != 0.0) ? a / fabs(s) : kInfD;
    d.prec_used[stage] = was_f64 ? 1 : 0;
    if (was_f64) {
      d.need_f64 = 0;
    } else {
      d.need_f64 = (d.fp64_kappa > 0.0 && d.kappa[stage] > d.fp64_kappa) ? 1 : 0;
    }
  }
  plugin_step(d, next);
}

// By a block.  Grid point k of the column: explicit h_in[k], the
// paper's default (linear over sigma [h0/4, 4 h0] = h_rot [1/4, 4]) or log-spaced
// over h_rot [lo, hi].  c32 = -log2(e) / (4 h^2), so exp2(D^2 c32) =
// exp(-D^2/(4 h^2)) and its square is exp(-D^2/(2 h^2)); c64 = -1/(4 h^2).
// Entries past n_h up to the chunk multiple hold -1 (finite, unused).
__device__ void lscv_prep(const ColDesc& c, double hr, int hc) {
  const int m = c.n_chunks * hc;
  for (int k = threadIdx.x; k < m; k += kThreads) {
    const int o = k;
    if (k < c.n_h) {
      double h;
      const double t = (c.n_h == 1) ? 0.0 : (double)k / (double)(c.n_h - 1);
      if (c.grid_kind == kGridExplicit)
        h = c.h_in[o];
      else if (c.grid_kind == kGridPaper)
        h = hr * 0.25 + (hr * 4.0 - hr * 0.25) * t;
      else
        h = hr * exp(log(c.grid_lo) + (log(c.grid_hi) - log(c.grid_lo)) * t);
      c.h[o] = h;
      const double q = 1.0 / (4.0 * h * h);
      c.c32[o] = (float)(-kLog2E * q);
      c.c64[o] = -q;
    } else {
      c.h[o] = 0.0;
      c.c32[o] = -1.0f;
      c.c64[o] = -1.0;
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_lscv_prep(const ColDesc* __restrict__ cols,
                                                        const int* __restrict__ ids, int hc) {
  const ColDesc c = cols[ids[blockIdx.x]];
  if (c.n_h > 0) lscv_prep(c, c.st->h_rot, hc);
}

// Spread and normal-reference bandwidth; then, where they follow at once, the
// first plug-in step (next) and the bandwidth grid (hc > 0).
__device__ void stats_final(const ColDesc& c, int next, int hc) {
  const int nblk = stat_blocks(c.n);
  __shared__ double sh[kThreads];
  __shared__ float shm[2 * kThreads];
  double s = 0.0;
  float lo = kInfF, hi = -kInfF;
  for (int b = threadIdx.x; b < nblk; b += kThreads) {
    s += c.stat[b];
    lo = fminf(lo, c.stat_mm[b]);
    hi = fmaxf(hi, c.stat_mm[kStatBlocks + b]);
  }
  s = block_sum(s, sh);
  block_minmax(lo, hi, shm);
  if (threadIdx.x == 0) {
    DevState& d = *c.st;
    d.xmin = lo;
    d.xmax = hi;
    const double n = d.n;
    d.var = s / (n - 1.0);
    d.sigma = sqrt(d.var);
    // normal-reference rule: (4/3)^(1/5) sigma n^(-1/5)
    d.h_rot = pow(4.0 / 3.0, 0.2) * pow(n, -0.2) * d.sigma;
    if (d.status == kStOk && !(d.sigma > 0.0 && isfinite(d.sigma))) d.status = kStDegenerate;
    sh[0] = d.h_rot;
    plugin_step(d, next);
  }
  if (hc > 0 && c.n_h > 0) {
    __syncthreads();
    lscv_prep(c, sh[0], hc);
  }
}

// Grids (max blocks, columns) for the passes over the samples, (columns) else.
__global__ __launch_bounds__(kThreads) void k_stats_sum(const ColDesc* __restrict__ cols, const int* __restrict__ ids) {
  stats_sum(cols[ids[blockIdx.y]], blockIdx.x);
}
__global__ __launch_bounds__(kThreads) void k_stats_mean(const ColDesc* __restrict__ cols,
                                                         const int* __restrict__ ids) {
  stats_mean(cols[ids[blockIdx.x]]);
}
__global__ __launch_bounds__(kThreads) void k_stats_dev(const ColDesc* __restrict__ cols, const int* __restrict__ ids) {
  stats_dev(cols[ids[blockIdx.y]], blockIdx.x);
}
__global__ __launch_bounds__(kThreads) void k_stats_final(const ColDesc* __restrict__ cols,
                                                          const int* __restrict__ ids, int next, int hc) {
  stats_final(cols[ids[blockIdx.x]], next, hc);
}

// Columns of one statistics block each (n <= 2048): the four passes by that
// block, in one launch.  A call of 1000 samples 138 -> 132 us.
__global__ __launch_bounds__(kThreads) void k_stats_one(const ColDesc* __restrict__ cols, const int* __restrict__ ids,
                                                        int next, int hc) {
  const ColDesc c = cols[ids[blockIdx.x]];
  stats_sum(c, 0);
  __syncthreads();
  stats_mean(c);
  __syncthreads();
  stats_dev(c, 0);
  __syncthreads();
  stats_final(c, next, hc);
}

// Where a sweep over j ends: its range, cut to the runs of kRun that hold a
// sample (what lies beyond n is padding and adds exact zeros).
__device__ __forceinline__ int sweep_end(int j_end, int n) { return min(j_end, (n + kRun - 1) / kRun * kRun); }
__device__ __forceinline__ int unit_end(const Unit& u, int n) { return sweep_end(u.j_end, n); }

// Samples j of an LSCV unit that share a partial-sum slot: a whole item of a
// column cut into pieces has a slot a piece, and its unit sweeps them one
// after the other, each from cleared sums, so that a slot holds the same bits
// as from a unit of its own.
__device__ __forceinline__ int slot_step(const Unit& u, const ColDesc& c) {
  return c.lscv_piece ? c.lscv_piece : u.j_end - u.j_begin;
}

// ------------------------------------------------------------------ psi pair kernels
// Mixed form.  The samples are pre-scaled by 1/g (y = x / g, one O(n) pass
// per stage), so a pair's w = u^2 = (y_i - y_j)^2 needs no per-pair scaling;
// the term He_r(u) e^(-u^2/2) is formed as He_r in w (Horner, the integer
// coefficients exact in FP32) times exp2(w * kPsiExp2), and both the term
// and its absolute value are accumulated by one fma each (|He_r| as a source
// modifier).  Per pair: sub, mul, mul, exp2, r/2 Horner ops, 2 fma.
// MASK (a wave's diagonal run): pairs with j <= i get w = kWMax, whose
// exponential is exactly 0 and whose He_r is finite.  CLAMP (padded tiles,
// or a column whose scaled range could overflow He_r): w = min(w, kWMax),
// so an infinite or huge distance also gives exactly 0.
// Bound: vector issue, as the LSCV sweep (see lscv_quad); the pairs of one
// LDS read go together: their exponentials at raised priority, then their
// polynomials and sums in pair order, which the plain work of other waves
// pairs with.  At n = 5e5 against one pair at a time: r = 8 24.8 -> 23.6 ms,
// r = 6 21.8 -> 20.5, r = 4 19.5 -> 18.8 (29.7, 25.8, 23.6 cycles a pair;
// 8.1 for the exponential and 2.4 for each of 9, 8, 7 plain instructions),
// the sums bitwise unchanged.
template <int R, bool MASK, bool CLAMP>
__device__ __forceinline__ void psi_run(const float4* __restrict__ run, int jg, float yi, int i, float& rs, float& ra) {
  rs = ra = 0.f;
#pragma unroll 4
  for (int q = 0; q < kRun / 4; ++q) {
    const float4 v = run[q];
    const float ys[4] = {v.x, v.y, v.z, v.w};
    float w[4], e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float d = yi - ys[u];
      w[u] = d * d;
      if (CLAMP) w[u] = fminf(w[u], kWMax);
      if (MASK) w[u] = (jg + 4 * q + u > i) ? w[u] : kWMax;
      e[u] = w[u] * kPsiExp2;
    }
    exp2_group(e);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float hw = herm_w<R>(w[u]);
      rs = __builtin_fmaf(hw, e[u], rs);
      ra = __builtin_fmaf(fabsf(hw), e[u], ra);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A psi unit of a large column: a row of 256 samples i, one per lane, against
// the unit's j-range.
template <int R>
__global__ __launch_bounds__(kThreads) void k_psi_units_f32(const ColDesc* __restrict__ cols,
                                                            const Unit* __restrict__ units, int u0) {
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (!c.st->active) return;
  const float* y = c.y32;
  const int n = c.n;
  const bool fast = c.st->psi_fast != 0;
  __shared__ float4 tile[kBJ / 4];
  __shared__ double red[2][4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = u.row * kBI;
  const int i = row0 + tid;
  const float yi = (i < n) ? y[i] : 0.f;
  const int wave_i0 = row0 + wave * 64;
  float aS = 0.f, cS = 0.f, aA = 0.f, cA = 0.f, rs, ra;
  const int j_end = unit_end(u, n);
  for (int t0 = u.j_begin; t0 < j_end; t0 += kBJ) {
    const int te = min(t0 + kBJ, j_end);
    __syncthreads();
    for (int q = tid; q < (te - t0) / 4; q += kThreads) tile[q] = reinterpret_cast<const float4*>(y + t0)[q];
    __syncthreads();
    int js = max(t0, wave_i0);
    if (js < te) {
      // uniform: unsafe range, or the tile holds padding (the two forms round
      // their polynomials differently, so the choice goes by whole tiles)
      const bool clamp = !fast || t0 + kBJ > n;
      if (js == wave_i0) {
        if (clamp)
          psi_run<R, true, true>(tile + (js - t0) / 4, js, yi, i, rs, ra);
        else
          psi_run<R, true, false>(tile + (js - t0) / 4, js, yi, i, rs, ra);
        kahan_add(aS, cS, rs);
        kahan_add(aA, cA, ra);
        js += kRun;
      }
      for (; js < te; js += kRun) {
        if (clamp)
          psi_run<R, false, true>(tile + (js - t0) / 4, js, yi, i, rs, ra);
        else
          psi_run<R, false, false>(tile + (js - t0) / 4, js, yi, i, rs, ra);
        kahan_add(aS, cS, rs);
        kahan_add(aA, cA, ra);
      }
    }
  }
  const bool valid = i < n;
  const double v = wave_sum2(valid ? (double)aS - (double)cS : 0.0, valid ? (double)aA - (double)cA : 0.0);
  if ((lane & 31) == 0) red[lane >> 5][wave] = v;
  __syncthreads();
  if (tid < 2)
    c.psi_part[(int64_t)tid * c.n_items_psi + u.item] = ((red[tid][0] + red[tid][1]) + red[tid][2]) + red[tid][3];
}

// A psi unit of a smaller column: 64 samples i (one per lane of every wave)
// against the unit's j-range, by the 16 waves of a block.  A tile holds
// 16 runs of 64 j, one a wave; the waves leave their runs' sums in LDS and
// waves 0 and 1 fold them, run by run in ascending j, into the lane's
// compensated sums of He e and |He| e while the next tile is swept.  The
// folds are those of one wave walking the whole j-range, as in the kernel
// above, so the two agree bitwise a lane; a j-range cut into more units would
// not do (the compensated sum depends on its grouping: psi moved by up to
// 4e-8 at kappa = 1000).  Bound: vector issue (psi_run).  With 256 samples i
// a block a column of n = 1000 had 4 blocks of 4 waves, one of n = 1e5 3
// waves a SIMD and a long last round.  A stage of r = 6 at n = 1000 36 -> 7
// us, at n = 12345 350 -> 47 us, at n = 1e5 1297 -> 977 us; eight waves a
// block take a call 2% longer at n = 5e3 to 1.2e4, four 14%; at n = 5e5 the
// 256-sample kernel is 4% faster (a barrier every 512 j against 64 j a wave).
constexpr int kPsiWaves = kPsiThreads / 64;
constexpr int kPsiTile = kPsiWaves * kRun;

template <int R>
__global__ __launch_bounds__(kPsiThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_psi_wide_f32(
    const ColDesc* __restrict__ cols, const Unit* __restrict__ units, int u0) {
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (!c.st->active) return;
  const float* x = c.x32;
  const float scale = c.st->psi_scale;
  const int n = c.n;
  const bool fast = c.st->psi_fast != 0;
  __shared__ __attribute__((aligned(16))) float tile[2][kPsiTile];
  __shared__ float part[2][2][kPsiWaves][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i0 = u.row * 64;
  const int i = i0 + lane;
  // rounded products, as in the scaled copy (padding: +inf, or NaN times a
  // scale of 0, which the clamp of padded tiles takes as far away)
  const auto y = [&](int j) {
#pragma clang fp contract(off)
    float v = x[j] * scale;
    asm volatile("" : "+v"(v));
    return v;
  };
  const float yi = (i < n) ? y(i) : 0.f;
  const int j_begin = max(u.j_begin, i0), j_end = unit_end(u, n);
  float acc = 0.f, comp = 0.f;  // waves 0 and 1: the lane's folded sums
  if (j_begin + tid < j_end) tile[0][tid] = y(j_begin + tid);
  __syncthreads();
  for (int t0 = j_begin, b = 0; t0 < j_end; t0 += kPsiTile, b ^= 1) {
    const int jn = t0 + kPsiTile + tid;
    float next = 0.f;
    if (jn < j_end) next = y(jn);
    const int js = t0 + wave * kRun;
    if (js < j_end) {
      const float4* run = reinterpret_cast<const float4*>(&tile[b][wave * kRun]);
      // the kBJ tile that the kernel above would hold the run in
      const bool clamp = !fast || js - ((js - u.j_begin) & (kBJ - 1)) + kBJ > n;
      float rs, ra;
      if (js == i0) {
        if (clamp)
          psi_run<R, true, true>(run, js, yi, i, rs, ra);
        else
          psi_run<R, true, false>(run, js, yi, i, rs, ra);
      } else {
        if (clamp)
          psi_run<R, false, true>(run, js, yi, i, rs, ra);
        else
          psi_run<R, false, false>(run, js, yi, i, rs, ra);
      }
      part[b][0][wave][lane] = rs;
      part[b][1][wave][lane] = ra;
    }
    tile[b ^ 1][tid] = next;
    __syncthreads();
    if (wave < 2) {
      // read before the buffer's next use: the wave reaches the next barrier
      // only after these reads
      const int runs = min(kPsiWaves, (j_end - t0) / kRun);
      for (int r = 0; r < runs; ++r) kahan_add(acc, comp, part[b][wave][r][lane]);
    }
  }
  if (wave < 2) {
    const double v = (i < n) ? (double)acc - (double)comp : 0.0;
    const double s = wave_sum2(v, v);
    if (lane == 0) c.psi_part[(int64_t)wave * c.n_items_psi + u.item] = s;
  }
}

template <int R, bool MASK>
__device__ __forceinline__ void psi_run64(const double* __restrict__ run, int jg, double xi, int i,
                                          double ig2, double cg, double& s, double& a) {
#pragma unroll 4
  for (int q = 0; q < kRun; ++q) {
    const double d = xi - run[q];
    double t = d * d;
    if (MASK) t = (jg + q > i) ? t : kInfD;
    const double w = fmin(t * ig2, (double)kWMax);
    const double term = herm_w64<R>(w) * exp_cw(t * cg);
    s += term;
    a += fabs(term);
  }
}

// conditional: run only when the FP32 pass flagged this column's stage (mixed form).
template <int R>
__global__ __launch_bounds__(kThreads) void k_psi_units_f64(const ColDesc* __restrict__ cols,
                                                            const Unit* __restrict__ units, int u0,
                                                            int conditional) {
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (!c.st->active) return;
  if (conditional && !c.st->need_f64) return;
  const double* x = c.x64;
  const int n = c.n;
  __shared__ double tile[kBJ];
  __shared__ double red[2][4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = u.row * kBI;
  const int i = row0 + tid;
  const double xi = (i < n) ? x[i] : 0.0;
  const int wave_i0 = row0 + wave * 64;
  const double ig2 = c.st->cd[0], cg = c.st->cd[1];
  double s = 0.0, a = 0.0;
  const int j_end = unit_end(u, n);
  for (int t0 = u.j_begin; t0 < j_end; t0 += kBJ) {
    const int te = min(t0 + kBJ, j_end);
    __syncthreads();
    for (int q = tid; q < (te - t0) / 2; q += kThreads)
      reinterpret_cast<double2*>(tile)[q] = reinterpret_cast<const double2*>(x + t0)[q];
    __syncthreads();
    int js = max(t0, wave_i0);
    if (js < te) {
      if (js == wave_i0) {
        psi_run64<R, true>(tile + js - t0, js, xi, i, ig2, cg, s, a);
        js += kRun;
      }
      for (; js < te; js += kRun) psi_run64<R, false>(tile + js - t0, js, xi, i, ig2, cg, s, a);
    }
  }
  const bool valid = i < n;
  const double v = wave_sum2(valid ? s : 0.0, valid ? a : 0.0);
  if ((lane & 31) == 0) red[lane >> 5][wave] = v;
  __syncthreads();
  if (tid < 2)
    c.psi_part[(int64_t)tid * c.n_items_psi + u.item] = ((red[tid][0] + red[tid][1]) + red[tid][2]) + red[tid][3];
}

// The same in the geometry of k_psi_wide_f32; every wave keeps FP64 sums of
// its own runs.
template <int R>
__global__ __launch_bounds__(kPsiThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_psi_wide_f64(
    const ColDesc* __restrict__ cols, const Unit* __restrict__ units, int u0, int conditional) {
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (!c.st->active) return;
  if (conditional && !c.st->need_f64) return;
  const double* x = c.x64;
  const int n = c.n;
  __shared__ double tile[2][kPsiTile];
  __shared__ double red[2][kPsiWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i0 = u.row * 64;
  const int i = i0 + lane;
  const double xi = (i < n) ? x[i] : 0.0;
  const double ig2 = c.st->cd[0], cg = c.st->cd[1];
  const int j_begin = max(u.j_begin, i0), j_end = unit_end(u, n);
  double s = 0.0, a = 0.0;
  if (j_begin + tid < j_end) tile[0][tid] = x[j_begin + tid];
  __syncthreads();
  for (int t0 = j_begin, b = 0; t0 < j_end; t0 += kPsiTile, b ^= 1) {
    const int jn = t0 + kPsiTile + tid;
    double next = 0.0;
    if (jn < j_end) next = x[jn];
    const int js = t0 + wave * kRun;
    if (js < j_end) {
      if (js == i0)
        psi_run64<R, true>(&tile[b][wave * kRun], js, xi, i, ig2, cg, s, a);
      else
        psi_run64<R, false>(&tile[b][wave * kRun], js, xi, i, ig2, cg, s, a);
    }
    tile[b ^ 1][tid] = next;
    __syncthreads();
  }
  const double v = wave_sum2((i < n) ? s : 0.0, (i < n) ? a : 0.0);
  if ((lane & 31) == 0) red[lane >> 5][wave] = v;
  __syncthreads();
  if (tid < 2) {
    double sum = red[tid][0];
    for (int w = 1; w < kPsiWaves; ++w) sum += red[tid][w];
    c.psi_part[(int64_t)tid * c.n_items_psi + u.item] = sum;
  }
}

// ------------------------------------------------------------------ LSCV kernels
// Four consecutive j of a run (one float4 of the LDS tile) against the
// lane's sample, for the HC bandwidths.  FIRST: the run's first pair starts
// the plain sums (S1 = e, S2 = e e instead of adding them to zero: the same
// values, as e is never -0), which saves clearing 2 HC registers per run.
//
// Bound: vector issue.  On gfx950 v_exp_f32 holds a SIMD's vector issue for
// 8.1 cycles a wave; the plain FP32 instructions of two waves issue together
// (2.0 to 2.5 cycles each instead of 4.2) as long as both waves are between
// their exponentials.  So the terms go in groups of kExpGroup: their
// products, their exponentials back to back at raised priority (a wave
// leaves its exponentials behind quickly), then their sums, 2 kExpGroup + the
// next products of plain work in one stretch that other waves' plain work
// pairs with.  Cycles a term and SIMD, n = 1e5 x 256 bandwidths, HC = 16: one
// term at a time with its priority raised from the exponential to its sums
// 16.9; groups of 2 15.1; of 4 14.96; of 8 15.1; the same groups without
// raised priority 21.2, with the plain part raised instead 21.0.  Estimate
// from the parts: 8.1 + 3.125 plain at 2.0 + the runs' folds (0.27) = 14.6 (the
// persistent sweep of n = 1e6 takes 14.57).  A column
// of n = 1e5, 256 bandwidths: 138.2 -> 121.9 ms (9.26 -> 10.50e12 terms/s),
// every sum bitwise unchanged.
// K0: the first bandwidth taken (the pruned sweep leaves out small ones).
template <int HC, bool MASK, bool FIRST, int K0>
__device__ __forceinline__ void lscv_quad(const float4 v, int jg, float xi, int i, const float (&ck)[HC],
                                          float (&r1)[HC], float (&r2)[HC]) {
  const float xs[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float d = xi - xs[u];
    float t = d * d;
    if (MASK) t = (jg + u > i) ? t : kInfF;
#pragma unroll
    for (int k0 = K0; k0 < HC; k0 += kExpGroup) {
      float e[kExpGroup];
#pragma unroll
      for (int k = 0; k < kExpGroup; ++k) e[k] = t * ck[k0 + k];
      exp2_group(e);
#pragma unroll
      for (int k = 0; k < kExpGroup; ++k) {
        if (FIRST && u == 0) {
          r1[k0 + k] = e[k];
          r2[k0 + k] = e[k] * e[k];
        } else {
          r1[k0 + k] += e[k];
          r2[k0 + k] = __builtin_fmaf(e[k], e[k], r2[k0 + k]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int HC, bool MASK, int K0 = 0>
__device__ __forceinline__ void lscv_run(const float4* __restrict__ tile, int jl, int jg, float xi, int i,
                                         const float (&ck)[HC], double (&a1)[HC], double (&a2)[HC]) {
  float r1[HC], r2[HC];
  lscv_quad<HC, MASK, true, K0>(tile[jl >> 2], jg, xi, i, ck, r1, r2);
#pragma unroll 3
  for (int q = 1; q < kRun / 4; ++q)
    lscv_quad<HC, MASK, false, K0>(tile[(jl >> 2) + q], jg + 4 * q, xi, i, ck, r1, r2);
  // the run's sums into the lane's FP64 accumulators
#pragma unroll
  for (int k = K0; k < HC; ++k) {
    a1[k] += (double)r1[k];
    a2[k] += (double)r2[k];
  }
}

// One LSCV work unit of the vector-ALU sweep: the unit's row of 256 samples
// i against its j-range, for the HC bandwidths of its chunk; the block's
// FP64 partial sums go to the unit's own slots (slot_step).  TJ: samples per LDS tile
// (256, 512 or 1024; a unit's j-range is a multiple of kRun, so a tile may
// end partly full).  The tile size changes only how often the block stages
// and synchronises: every lane still folds its terms in runs of 64 j in
// ascending j order, so every (unit, h) sum is bitwise the same for all TJ.
template <int HC, int TJ>
__device__ __forceinline__ void lscv_unit_f32(const ColDesc* __restrict__ cols, const Unit& u, float4* tile,
                                              double (*red)[2 * HC]) {
  const ColDesc c = cols[u.col];
  if (c.st->status != kStOk) return;  // uniform over the block
  const float* x = c.x32;
  const int n = c.n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = u.row * kBI;
  const int i = row0 + tid;
  const float xi = (i < n) ? x[i] : 0.f;
  const int wave_i0 = row0 + wave * 64;
  const float* cc = c.c32 + u.chunk * HC;
  float ck[HC];
#pragma unroll
  for (int k = 0; k < HC; ++k) ck[k] = uniform_f32(cc[k]);
  const int step = slot_step(u, c);
  for (int p0 = u.j_begin, slot = u.item; p0 < u.j_end; p0 += step, ++slot) {
    if (p0 > u.j_begin) __syncthreads();  // red has been read
    double a1[HC], a2[HC];
#pragma unroll
    for (int k = 0; k < HC; ++k) a1[k] = a2[k] = 0.0;
    const int j_end = sweep_end(p0 + step, n);
    for (int t0 = p0; t0 < j_end; t0 += TJ) {
      const int te = min(t0 + TJ, j_end);
      __syncthreads();
      for (int q = tid; q < (te - t0) / 4; q += kThreads) tile[q] = reinterpret_cast<const float4*>(x + t0)[q];
      __syncthreads();
      int js = max(t0, wave_i0);
      if (js < te) {
        if (js == wave_i0) {
          lscv_run<HC, true>(tile, js - t0, js, xi, i, ck, a1, a2);
          js += kRun;
        }
        for (; js < te; js += kRun) lscv_run<HC, false>(tile, js - t0, js, xi, i, ck, a1, a2);
      }
    }
    const bool valid = i < n;
    double v[2 * HC];
#pragma unroll
    for (int k = 0; k < HC; ++k) {
      v[2 * k] = valid ? a1[k] : 0.0;
      v[2 * k + 1] = valid ? a2[k] : 0.0;
    }
    wave_sums(v, red[wave], lane);
    __syncthreads();
    if (tid < 2 * HC) {
      const int h = u.chunk * HC + (tid >> 1);
      if (h < c.n_h) {
        const double v = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
        c.part[(int64_t)(2 * h + (tid & 1)) * c.n_items + slot] = v;
      }
    }
  }
}

template <int HC>
__global__ __launch_bounds__(kThreads) void k_lscv_units_f32(const ColDesc* __restrict__ cols,
                                                             const Unit* __restrict__ units, int u0) {
  __shared__ float4 tile[kBJ / 4];
  __shared__ double red[4][2 * HC];
  lscv_unit_f32<HC, kBJ>(cols, units[u0 + blockIdx.x], tile, red);
}

// Persistent form: a grid of about as many blocks as the chip holds at once
// takes the pass's units from device counters, one unit per block at a time,
// until the list is exhausted.  The list comes in kQueueGroups groups of
// about equal work, each a contiguous stretch of (column, j) positions kept
// largest first; group g is units [group_begin[g], group_begin[g + 1]) with
// counter next[g].  Block b starts on group b % kQueueGroups (workgroups are
// dealt round-robin to the eight dies, so a die's blocks stream the sample
// tiles of one stretch of the column, which stays in that die's L2), and
// when its group is drained it moves on to the next ones, taking what is
// left there.  A block leaves a group once its counter passes the group's
// end, so every block reaches the end of the last group and exits.  One
// launch covers a whole pass; the longest units start first wherever a
// block frees up.  next[0 .. kQueueGroups) must be 0 at launch.
template <int HC, int TJ>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(HC <= 16 ? 4 : 2))) void
k_lscv_units_f32_queue(const ColDesc* __restrict__ cols, const Unit* __restrict__ units,
                       const int* __restrict__ group_begin, int* __restrict__ next) {
  __shared__ float4 tile[TJ / 4];
  __shared__ double red[4][2 * HC];
  __shared__ int cur;
  const int g0 = (int)(blockIdx.x % kQueueGroups);
  for (int q = 0; q < kQueueGroups; ++q) {
    const int g = (g0 + q) % kQueueGroups;
    const int base = group_begin[g], len = group_begin[g + 1] - base;
    for (;;) {
      if (threadIdx.x == 0) cur = atomicAdd(next + g, 1);
      __syncthreads();
      const int k = __builtin_amdgcn_readfirstlane(cur);  // uniform: unit and column loads stay scalar
      __syncthreads();
      if (k >= len) break;
      lscv_unit_f32<HC, TJ>(cols, units[base + k], tile, red);
    }
  }
}

// Clears n ints (the work counters of a pass) with a kernel, so the pass
// stays replayable from a graph.
__global__ void k_zero_ints(int* __restrict__ p, int n) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = 0;
}

// Reference rate of the sweep's inner loop on the part: lscv_run<HC, false> over
// one LDS tile of kBJ samples staged once, `reps` times per block, with no further
// staging, barriers, masks or partial-sum writes (each wave stores one sum so
// that nothing is dropped).  Evaluations per launch:
// blocks x kThreads x reps x kBJ x HC.
template <int HC>
__global__ __launch_bounds__(kThreads) void k_lscv_ceiling(const float* __restrict__ x, const float* __restrict__ c32,
                                                           int reps, double* __restrict__ out) {
  __shared__ float4 tile[kBJ / 4];
  const int tid = threadIdx.x;
  for (int q = tid; q < kBJ / 4; q += kThreads) tile[q] = reinterpret_cast<const float4*>(x)[q];
  __syncthreads();
  const float xi = x[tid] + 0.5f;
  float ck[HC];
  double a1[HC], a2[HC];
#pragma unroll
  for (int k = 0; k < HC; ++k) {
    ck[k] = uniform_f32(c32[k]);
    a1[k] = a2[k] = 0.0;
  }
  for (int r = 0; r < reps; ++r)
    for (int js = 0; js < kBJ; js += kRun) lscv_run<HC, false>(tile, js, js, xi, 0, ck, a1, a2);
  double v = 0.0;
#pragma unroll
  for (int k = 0; k < HC; ++k) v += (a1[k]) + (a2[k]);
  v = wave_sum(v);
  if ((tid & 63) == 0) out[(int64_t)blockIdx.x * (kThreads / 64) + (tid >> 6)] = v;
}

// Tile pruning (mixed form, sorted column): the squared distance D2 beyond
// which pairs of bandwidths [k0, k1) are skipped, 256 x 512 at a time or less.
// A skipped tile holds at most 2^17 pairs, each term at most exp2(c_max D^2)
// (c_max: the coefficient closest to zero, i.e. the largest h) for S1 and its
// square for S2.  With T an upper bound on the (row, tile) pairs of the column
// and L1, L2 the smallest near-tile sums (lower bounds of S1, S2: all terms
// are positive) over the bandwidths, pairs are skipped only when 2^17 exp2(c_max
// D^2) < eps L1 / T and 2^17 exp2(2 c_max D^2) < eps L2 / T, so everything
// skipped is below eps S1(h) and eps S2(h) for every h of them.
__device__ double prune_cut(const ColDesc& c, int k0, int k1, double eps) {
  const double n = (double)c.n;
  const double rows = ceil(n / kBI);
  const double T = rows * (ceil(n / kBJ) + 1.0);
  const double lt = log2(eps / (T * (double)kBI * (double)kBJ));
  double l1 = kInfD, l2 = kInfD, cmax = -kInfD;
  for (int k = k0; k < k1; ++k) {
    l1 = fmin(l1, c.near_sums[2 * k]);
    l2 = fmin(l2, c.near_sums[2 * k + 1]);
    cmax = fmax(cmax, (double)c.c32[k]);
  }
  if (!(l1 > 0.0 && l2 > 0.0 && cmax < 0.0)) return kInfD;
  const double d1 = (lt + log2(l1)) / cmax;
  const double d2 = (lt + log2(l2)) / (2.0 * cmax);
  return fmax(d1, d2) * (1.0 + 1e-6) + 1e-30;
}

// The cut of every bandwidth chunk of a column.
__global__ __launch_bounds__(kThreads) void k_lscv_prune_prep(const ColDesc* __restrict__ cols,
                                                              const int* __restrict__ ids, int hc, double eps) {
  const ColDesc c = cols[ids[blockIdx.x]];
  if (c.n_h <= 0 || c.st->status != kStOk) return;
  for (int ch = threadIdx.x; ch < c.n_chunks; ch += blockDim.x)
    c.d2cut[ch] = (float)prune_cut(c, ch * hc, min(c.n_h, (ch + 1) * hc), eps);
}

// Tile pruning on sorted samples: the same sweep over a column sorted
// ascending, whose j-tiles therefore lie at growing distance from the unit's
// row of i.  A uniform scan of the tiles' first samples finds the first tile
// whose smallest distance to the row exceeds the chunk's cut (every later
// tile is farther still); the sweep stops there.  Before that, each wave
// leaves out, run by run, the quarters of its chunk (half chunks of 8) whose
// own cuts lie nearer: a chunk of 16 of 128 bandwidths over [h_rot / 64, 4
// h_rot] spans a factor of two in h, and so in the distance that matters.
// All skipped pairs are counted exactly.  n = 150,001, bimodal, 128 bandwidths
// (dense 137 ms): the sweep with whole chunks 0.447 of the evaluations in 66.5
// ms, with parts 0.399 in 61 ms.
template <int HC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(HC <= 16 ? 4 : 2)))
void k_lscv_units_prune(const ColDesc* __restrict__ cols, const Unit* __restrict__ units, int u0, double eps) {
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (c.st->status != kStOk) return;
  const float* x = c.x32;
  const int n = c.n;
  const int row0 = u.row * kBI;
  int j_end = unit_end(u, n);
  {
    const float row_max = x[min(row0 + kBI, n) - 1];
    const float cut = c.d2cut[u.chunk];
    for (int t = u.j_begin; t < j_end; t += kBJ) {
      const float dd = x[t] - row_max;
      if (dd > 0.f && dd * dd > cut) {
        j_end = t;
        break;
      }
    }
  }
  constexpr int kParts = HC >= 16 ? 4 : HC / kExpGroup, kPart = HC / kParts;
  __shared__ float4 tile[kBJ / 4];
  __shared__ double red[4][2 * HC];
  __shared__ float part_cut[kParts];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = row0 + tid;
  const float xi = (i < n) ? x[i] : 0.f;
  const int wave_i0 = row0 + wave * 64;
  const float* cc = c.c32 + u.chunk * HC;
  float ck[HC];
  double a1[HC], a2[HC];
#pragma unroll
  for (int k = 0; k < HC; ++k) {
    ck[k] = uniform_f32(cc[k]);
    a1[k] = a2[k] = 0.0;
  }
  // a part with no bandwidth of the grid is always left out
  if (tid < kParts) {
    const int k0 = u.chunk * HC + tid * kPart, k1 = min(c.n_h, k0 + kPart);
    part_cut[tid] = k0 < k1 ? (float)prune_cut(c, k0, k1, eps) : -1.0f;
  }
  __syncthreads();
  float cut[kParts];
#pragma unroll
  for (int p = 0; p < kParts; ++p) cut[p] = uniform_f32(part_cut[p]);
  const float wave_max = x[min(wave_i0 + 64, n) - 1];
  const int wave_rows = max(0, min(64, n - wave_i0));
  const int wave_h = min(HC, c.n_h - u.chunk * HC);
  double skipped = 0.0;  // uniform over the wave
  for (int t0 = u.j_begin; t0 < j_end; t0 += kBJ) {
    const int te = min(t0 + kBJ, j_end);
    __syncthreads();
    for (int q = tid; q < (te - t0) / 4; q += kThreads) tile[q] = reinterpret_cast<const float4*>(x + t0)[q];
    __syncthreads();
    int js = max(t0, wave_i0);
    if (js < te) {
      if (js == wave_i0) {
        lscv_run<HC, true>(tile, js - t0, js, xi, i, ck, a1, a2);
        js += kRun;
      }
      for (; js < te; js += kRun) {
        // the first part of the chunk that the run's nearest pair is within
        // the cut of (later parts hold larger bandwidths)
        const float dd = fmaxf(uniform_f32(reinterpret_cast<const float*>(tile)[js - t0]) - wave_max, 0.f);
        int p = 0;
        while (p < kParts && dd * dd > cut[p]) ++p;
        if (p) skipped += (double)wave_rows * (double)(min(js + kRun, n) - js) * (double)min(p * kPart, wave_h);
        if (p == 0)
          lscv_run<HC, false>(tile, js - t0, js, xi, i, ck, a1, a2);
        else if (p == 1 && kParts > 1)
          lscv_run<HC, false, kPart % HC>(tile, js - t0, js, xi, i, ck, a1, a2);
        else if (p == 2 && kParts > 2)
          lscv_run<HC, false, 2 * kPart % HC>(tile, js - t0, js, xi, i, ck, a1, a2);
        else if (p == 3 && kParts > 3)
          lscv_run<HC, false, 3 * kPart % HC>(tile, js - t0, js, xi, i, ck, a1, a2);
      }
    }
  }
  if (lane == 0 && skipped > 0.0) atomicAdd(&c.st->pruned_evals, skipped);
  if (tid == 0 && j_end < u.j_end && j_end < n) {
    // every skipped tile lies right of the row (distance > 0): all its pairs count
    const double rows = (double)min(kBI, n - row0);
    const double hv = (double)min(HC, c.n_h - u.chunk * HC);
    atomicAdd(&c.st->pruned_evals, rows * (double)(min(u.j_end, n) - j_end) * hv);
  }
  const bool valid = i < n;
  double v[2 * HC];
#pragma unroll
  for (int k = 0; k < HC; ++k) {
    v[2 * k] = valid ? a1[k] : 0.0;
    v[2 * k + 1] = valid ? a2[k] : 0.0;
  }
  wave_sums(v, red[wave], lane);
  __syncthreads();
  if (tid < 2 * HC) {
    const int h = u.chunk * HC + (tid >> 1);
    if (h < c.n_h) {
      const double v = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
      c.part[(int64_t)(2 * h + (tid & 1)) * c.n_items + u.item] = v;
    }
  }
}

// 2^(j / 64), j = 0 .. 63: the low and high words of the nearest double, and the
// high word of what that leaves (evaluated in 60 digits).
__constant__ uint32_t kExp2Tab[3][64] = {
    {
     0x00000000u, 0x3e778061u, 0xd3158574u, 0x18759bc8u, 0x6cf9890fu, 0x32d3d1a2u, 0xd0125b51u, 0xaea92de0u,
     0x3c7d517bu, 0xeb6fcb75u, 0x3168b9aau, 0x88628cd6u, 0x6e756238u, 0x65e27cddu, 0xf51fdee1u, 0xa6e4030bu,
     0x0a31b715u, 0xb26416ffu, 0x373aa9cbu, 0x34e59ff7u, 0x4c123422u, 0x21f72e2au, 0x6061892du, 0xb5c13cd0u,
     0xd5362a27u, 0x769d2ca7u, 0x569d4f82u, 0x36b527dau, 0xdd485429u, 0x15ad2148u, 0xb03a5585u, 0x82552225u,
     0x667f3bcdu, 0x3c651a2fu, 0xe8ec5f74u, 0x564267c9u, 0x73eb0187u, 0x36cf4e62u, 0x994cce13u, 0x9b4492edu,
     0x422aa0dbu, 0x99157736u, 0xb0cdc5e5u, 0x9fde4e50u, 0x82a3f090u, 0x7b5de565u, 0xb23e255du, 0x5579fdbfu,
     0x995ad3adu, 0xb84f15fbu, 0xf2fb5e47u, 0x904bc1d2u, 0xdd85529cu, 0x2e57d14bu, 0xdcef9069u, 0x4a07897cu,
     0xdcfba487u, 0x03db3285u, 0x337b9b5fu, 0xe78b3ff6u, 0xa2a490dau, 0xee615a27u, 0x5b6e4540u, 0x819e90d8u,
    },
    {
     0x3ff00000u, 0x3ff02c9au, 0x3ff059b0u, 0x3ff08745u, 0x3ff0b558u, 0x3ff0e3ecu, 0x3ff11301u, 0x3ff1429au,
     0x3ff172b8u, 0x3ff1a35bu, 0x3ff1d487u, 0x3ff2063bu, 0x3ff2387au, 0x3ff26b45u, 0x3ff29e9du, 0x3ff2d285u,
     0x3ff306feu, 0x3ff33c08u, 0x3ff371a7u, 0x3ff3a7dbu, 0x3ff3dea6u, 0x3ff4160au, 0x3ff44e08u, 0x3ff486a2u,
     0x3ff4bfdau, 0x3ff4f9b2u, 0x3ff5342bu, 0x3ff56f47u, 0x3ff5ab07u, 0x3ff5e76fu, 0x3ff6247eu, 0x3ff66238u,
     0x3ff6a09eu, 0x3ff6dfb2u, 0x3ff71f75u, 0x3ff75febu, 0x3ff7a114u, 0x3ff7e2f3u, 0x3ff82589u, 0x3ff868d9u,
     0x3ff8ace5u, 0x3ff8f1aeu, 0x3ff93737u, 0x3ff97d82u, 0x3ff9c491u, 0x3ffa0c66u, 0x3ffa5503u, 0x3ffa9e6bu,
     0x3ffae89fu, 0x3ffb33a2u, 0x3ffb7f76u, 0x3ffbcc1eu, 0x3ffc199bu, 0x3ffc67f1u, 0x3ffcb720u, 0x3ffd072du,
     0x3ffd5818u, 0x3ffda9e6u, 0x3ffdfc97u, 0x3ffe502eu, 0x3ffea4afu, 0x3ffefa1bu, 0x3fff5076u, 0x3fffa7c1u,
    },
    {
     0x00000000u, 0xbc719083u, 0x3c8d73e3u, 0x3c6186beu, 0x3c98a62eu, 0x3c403a17u, 0xbc96c510u, 0xbc932fc0u,
     0xbc819042u, 0x3c8e5b4cu, 0x3c9e016eu, 0x3c8dc776u, 0x3c99b07fu, 0x3c82bd34u, 0x3c8612e9u, 0x3c900247u,
     0x3c86f46bu, 0x3c932722u, 0xbc963aebu, 0xbc75e437u, 0x3c8ada09u, 0xbc5ef369u, 0x3c489b7au, 0x3c73c1a4u,
     0x3c7d4398u, 0xbc94b30au, 0xbc807abeu, 0x3c99bb2cu, 0x3c96324cu, 0x3c9ba6f9u, 0xbc9383c1u, 0xbc9bb60au,
     0xbc9bdd34u, 0xbc6bbe3au, 0xbc816e48u, 0xbc902459u, 0xbc841578u, 0x3c705d03u, 0xbc9d4c1eu, 0xbc9fc6f9u,
     0x3c96e9f1u, 0x3c85cc14u, 0xbc675fc8u, 0xbc9d185bu, 0x3c7c7c47u, 0xbc935949u, 0xbc9d2f6fu, 0x3c90fac9u,
     0x3c97a1cdu, 0xbc62805eu, 0xbc75584fu, 0x3c823dd0u, 0x3c811066u, 0x3c92884eu, 0x3c7503ccu, 0xbc9cbc37u,
     0x3c82ed03u, 0x3c9c2300u, 0xbc91a5cdu, 0x3c839e8au, 0xbc9e9c23u, 0x3c9dc7f5u, 0x3c99d3e1u, 0x3c874854u,
    },
};

// exp_cw's e^x with |r| <= ln(2) / 128, by the table method of Tang (ACM Trans.
// Math. Softw. 15, 1989): e^x = 2^(n >> 6) (T + T (r + r^2 q(r))),
// T = 2^((n & 63) / 64) from the words of kExp2Tab in LDS (a row's 64 words lie
// in 64 banks, so that lanes that differ read different banks), q of degree 3
// with least maximal relative error in e^r (1.4e-18).  13 FP64 instructions
// instead of 18, with 4 integer ones that cost half; error over [-708, 0], in
// 2^-53: at most 1.02, 0.359 on average (exp_cw: 1.23 and 0.369).
// n = 12345 x 150 bandwidths 8.36 -> 7.97 ms: FP64 at its issue rate draws the
// clock down to 1.9 GHz, so the time follows the work, not its latency (four
// waves a SIMD instead of three change nothing).
__device__ __forceinline__ double exp_tab(double x, const uint32_t* tab) {
  constexpr double kScale = 92.33248261689366;      // 64 / ln 2
  constexpr double kHead = 0x1.62e42ff000000p-7;   // ln 2 / 64 rounded to 33 bits
  constexpr double kTail = -6.563929801064195e-13;  // ln 2 / 64 - head
  constexpr double kRound = 0x1.8p52;
  x = fmax(x, -1100.0);
  const double t = __builtin_fma(x, kScale, kRound);
  const double k = t - kRound;
  double r = __builtin_fma(-k, kHead, x);
  r = __builtin_fma(-k, kTail, r);
  const uint32_t n = (uint32_t)__builtin_bit_cast(uint64_t, t), j = n & 63;
  const double T = __builtin_bit_cast(double, (uint64_t)tab[64 + j] << 32 | tab[j]);
  const double tail = __builtin_bit_cast(double, (uint64_t)tab[128 + j] << 32);
  double q = 0.008333334352148097;
  q = __builtin_fma(q, r, 0.04166672338953993);
  q = __builtin_fma(q, r, 0.1666666666667746);
  q = __builtin_fma(q, r, 0.4999999999994852);
  const double s = __builtin_fma(r * r, q, r);
  return ldexp(T + __builtin_fma(T, s, tail), (int)n >> 6);
}

template <int HC, bool MASK>
__device__ __forceinline__ void lscv_run64(const double* __restrict__ tile, int jl, int jg, double xi, int i,
                                           const double (&ck)[HC], const uint32_t* tab, double (&s1)[HC],
                                           double (&s2)[HC]) {
#pragma unroll 2
  for (int q = 0; q < kRun; ++q) {
    const double d = xi - tile[jl + q];
    double t = d * d;
    if (MASK) t = (jg + q > i) ? t : kInfD;
#pragma unroll
    for (int k = 0; k < HC; ++k) {
      const double e = exp_tab(t * ck[k], tab);
      s1[k] += e;
      s2[k] = __builtin_fma(e, e, s2[k]);
    }
  }
}

template <int HC>
__global__ __launch_bounds__(kThreads) void k_lscv_units_f64(const ColDesc* __restrict__ cols,
                                                             const Unit* __restrict__ units, int u0) {
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (c.st->status != kStOk) return;
  const double* x = c.x64;
  const int n = c.n;
  __shared__ double tile[kBJ];
  __shared__ uint32_t tab[3 * 64];
  __shared__ double red[4][2 * HC];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = u.row * kBI;
  const int i = row0 + tid;
  const double xi = (i < n) ? x[i] : 0.0;
  const int wave_i0 = row0 + wave * 64;
  const double* cc = c.c64 + u.chunk * HC;
  double ck[HC];
#pragma unroll
  for (int k = 0; k < HC; ++k) ck[k] = cc[k];
  if (tid < 3 * 64) tab[tid] = kExp2Tab[0][tid];
  const int step = slot_step(u, c);
  for (int p0 = u.j_begin, slot = u.item; p0 < u.j_end; p0 += step, ++slot) {
    if (p0 > u.j_begin) __syncthreads();  // red has been read
    double s1[HC], s2[HC];
#pragma unroll
    for (int k = 0; k < HC; ++k) s1[k] = s2[k] = 0.0;
    const int j_end = sweep_end(p0 + step, n);
    for (int t0 = p0; t0 < j_end; t0 += kBJ) {
      const int te = min(t0 + kBJ, j_end);
      __syncthreads();
      for (int q = tid; q < (te - t0) / 2; q += kThreads)
        reinterpret_cast<double2*>(tile)[q] = reinterpret_cast<const double2*>(x + t0)[q];
      __syncthreads();
      int js = max(t0, wave_i0);
      if (js < te) {
        if (js == wave_i0) {
          lscv_run64<HC, true>(tile, js - t0, js, xi, i, ck, tab, s1, s2);
          js += kRun;
        }
        for (; js < te; js += kRun) lscv_run64<HC, false>(tile, js - t0, js, xi, i, ck, tab, s1, s2);
      }
    }
    const bool valid = i < n;
    double v[2 * HC];
#pragma unroll
    for (int k = 0; k < HC; ++k) {
      v[2 * k] = valid ? s1[k] : 0.0;
      v[2 * k + 1] = valid ? s2[k] : 0.0;
    }
    wave_sums(v, red[wave], lane);
    __syncthreads();
    if (tid < 2 * HC) {
      const int h = u.chunk * HC + (tid >> 1);
      if (h < c.n_h) {
        const double v = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
        c.part[(int64_t)(2 * h + (tid & 1)) * c.n_items + slot] = v;
      }
    }
  }
}

// ---- LSCV pair kernel with the exponent arguments formed on the matrix cores.
// The argument of every (pair, h) term is D^2 * c_h: an outer product of the
// pair distances and the chunk's coefficients.  v_mfma_f32_32x32x2f32 forms
// it for 32 samples i x 2 samples j x 16 bandwidths at once (A[row][k] =
// D^2(i_row, j_k), B[k][col] = c[col % 16] if k = col / 16 else 0), so the
// vector ALU only evaluates exp2 and accumulates.  Lane l ends up owning
// bandwidth h = l % 16 for rows 8(r/4) + 4(l/32) + r%4 of the output block.
// Groups of 16 j whose pairs are all valid (j > i, i < n, j < n) run without
// masks; the others replace the argument of an invalid pair by -inf.
typedef float v16f __attribute__((ext_vector_type(16)));
constexpr float kBigF = 3.0e38f;

template <bool MASK>
__device__ __forceinline__ void mfma_consume(const v16f& da, const v16f& db, int j0, int jsel, int k, int ibase,
                                             int n, float (&s1)[4], float (&s2)[4]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float ya = da[r], yb = db[r];
    if (MASK) {
      const int row = 8 * (r >> 2) + 4 * k + (r & 3);
      const int j = j0 + jsel;
      const int ia = ibase + row, ib = ibase + 32 + row;
      ya = (j > ia && ia < n && j < n) ? ya : -kInfF;
      yb = (j > ib && ib < n && j < n) ? yb : -kInfF;
    }
    const float ea = __builtin_amdgcn_exp2f(ya);
    const float eb = __builtin_amdgcn_exp2f(yb);
    s1[r & 3] += ea;
    s2[r & 3] = __builtin_fmaf(ea, ea, s2[r & 3]);
    s1[r & 3] += eb;
    s2[r & 3] = __builtin_fmaf(eb, eb, s2[r & 3]);
  }
}

// 8 pairs (j, j+1) of one group of 16 j; the matrix-core products of the next
// pair are issued before the exponentials of the current one.
template <bool MASK>
__device__ __forceinline__ void mfma_group(const float4* __restrict__ tile, int jl, int jg, float xa, float xb,
                                           int ibase, int n, float bop, int lane, float (&s1)[4], float (&s2)[4]) {
  const int k = lane >> 5;
  const int jsel = (lane & 31) >> 4;
  const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float xj[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = tile[(jl >> 2) + q];
    xj[2 * q] = k ? v.y : v.x;
    xj[2 * q + 1] = k ? v.w : v.z;
  }
  float ta = xa - xj[0], tb = xb - xj[0];
  v16f da = __builtin_amdgcn_mfma_f32_32x32x2f32(fminf(ta * ta, kBigF), bop, zero, 0, 0, 0);
  v16f db = __builtin_amdgcn_mfma_f32_32x32x2f32(fminf(tb * tb, kBigF), bop, zero, 0, 0, 0);
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    v16f na, nb;
    if (p < 7) {
      ta = xa - xj[p + 1];
      tb = xb - xj[p + 1];
      na = __builtin_amdgcn_mfma_f32_32x32x2f32(fminf(ta * ta, kBigF), bop, zero, 0, 0, 0);
      nb = __builtin_amdgcn_mfma_f32_32x32x2f32(fminf(tb * tb, kBigF), bop, zero, 0, 0, 0);
    }
    mfma_consume<MASK>(da, db, jg + 2 * p, jsel, k, ibase, n, s1, s2);
    if (p < 7) {
      da = na;
      db = nb;
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_lscv_units_mfma(const ColDesc* __restrict__ cols,
                                                              const Unit* __restrict__ units, int u0) {
  constexpr int HC = 16;
  const Unit u = units[u0 + blockIdx.x];
  const ColDesc c = cols[u.col];
  if (c.st->status != kStOk) return;
  const float* x = c.x32;
  const int n = c.n;
  __shared__ float4 tile[kBJ / 4];
  __shared__ double red[4][HC][2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = u.row * kBI;
  const int wave_i0 = row0 + wave * 64;
  // A-operand rows: lane l holds samples i = wave_i0 + (l % 32) and i + 32
  const int ia = wave_i0 + (lane & 31), ib = ia + 32;
  const float xa = (ia < n) ? x[ia] : 0.f;
  const float xb = (ib < n) ? x[ib] : 0.f;
  // B operand: k = lane / 32, col = lane % 32
  const int kb = lane >> 5, colb = lane & 31;
  const float bop = (kb == (colb >> 4)) ? c.c32[u.chunk * HC + (colb & 15)] : 0.f;
  const bool rows_full = wave_i0 + 64 <= n;
  const int step = slot_step(u, c);
  for (int p0 = u.j_begin, slot = u.item; p0 < u.j_end; p0 += step, ++slot) {
    if (p0 > u.j_begin) __syncthreads();  // red has been read
    float a1 = 0.f, c1 = 0.f, a2 = 0.f, c2 = 0.f;
    const int j_end = sweep_end(p0 + step, n);
    for (int t0 = p0; t0 < j_end; t0 += kBJ) {
      const int te = min(t0 + kBJ, j_end);
      __syncthreads();
      for (int q = tid; q < (te - t0) / 4; q += kThreads) tile[q] = reinterpret_cast<const float4*>(x + t0)[q];
      __syncthreads();
      for (int js = max(t0, wave_i0); js < te; js += 16) {
        float s1[4] = {0.f, 0.f, 0.f, 0.f}, s2[4] = {0.f, 0.f, 0.f, 0.f};
        const bool clean = rows_full && js >= wave_i0 + 64 && js + 16 <= n;
        if (clean)
          mfma_group<false>(tile, js - t0, js, xa, xb, wave_i0, n, bop, lane, s1, s2);
        else
          mfma_group<true>(tile, js - t0, js, xa, xb, wave_i0, n, bop, lane, s1, s2);
        kahan_add(a1, c1, (s1[0] + s1[1]) + (s1[2] + s1[3]));
        kahan_add(a2, c2, (s2[0] + s2[1]) + (s2[2] + s2[3]));
      }
    }
    // lanes l, l^16, l^32, l^48 hold the same bandwidth
    double v1 = (double)a1 - (double)c1, v2 = (double)a2 - (double)c2;
    v1 += __shfl_xor(v1, 16, 64);
    v2 += __shfl_xor(v2, 16, 64);
    v1 += __shfl_xor(v1, 32, 64);
    v2 += __shfl_xor(v2, 32, 64);
    if (lane < HC) {
      red[wave][lane][0] = v1;
      red[wave][lane][1] = v2;
    }
    __syncthreads();
    if (tid < 2 * HC) {
      const int hk = tid >> 1, w = tid & 1;
      const int h = u.chunk * HC + hk;
      if (h < c.n_h) {
        const double v = ((red[0][hk][w] + red[1][hk][w]) + red[2][hk][w]) + red[3][hk][w];
        c.part[(int64_t)(2 * h + w) * c.n_items + slot] = v;
      }
    }
  }
}

// Block per column.  g(h) = h^-1 [2 n^-2 ((4pi)^-1/2 S1 - 2 (2pi)^-1/2 S2) + n^-1 (4pi)^-1/2];
// gscale with +.  Grid argmin with ties to the lowest index.
// g(h) of every grid point, argmin, edge flag and margin.  The mixed form's
// pair sums are exact sums at the bandwidth whose FP32 exponent coefficient
// c32 = -log2(e)/(4 h^2) is exactly representable; that bandwidth (within
// 3e-8 of the grid value) also goes into the 1/h factor, so each g is a
// consistent evaluation at a point next to the grid value rather than a
// mixture of two bandwidths, and the per-point error does not jump from one
// grid point to the next with the rounding of its coefficient.
__global__ __launch_bounds__(1024) void k_lscv_finalize(const ColDesc* __restrict__ cols,
                                                        const int* __restrict__ ids, int f64) {
  const ColDesc c = cols[ids[blockIdx.x]];
  if (c.n_h <= 0) return;
  DevState& d = *c.st;
  const int n_h = c.n_h;
  const double* sums = c.sums;
  const double* h_dev = c.h;
  double* g = c.g;
  double* gscale = c.gs;
  __shared__ double bv[1024];
  __shared__ int bk[1024];
  const int t = threadIdx.x;
  const double n = d.n;
  const double ckk = 1.0 / sqrt(4.0 * kPi), ck = 1.0 / sqrt(2.0 * kPi);
  const bool ok = d.status == kStOk;
  double best = kInfD;
  int kbest = 0x7fffffff;
  for (int k = t; k < n_h; k += blockDim.x) {
    const double s1 = sums[2 * k], s2 = sums[2 * k + 1];
    double h = h_dev[k];
    if (!f64) {
      const double cq = (double)c.c32[k];
      if (cq < 0.0 && isfinite(cq)) h = sqrt(-kLog2E / (4.0 * cq));
    }
    const double a = ckk * s1, b = ck * s2;
    const double gv = (2.0 / (n * n) * (a - 2.0 * b) + ckk / n) / h;
    g[k] = ok ? gv : NAN;
    gscale[k] = ok ? (2.0 / (n * n) * (a + 2.0 * b) + ckk / n) / h : NAN;
    if (gv < best) {
      best = gv;
      kbest = k;
    }
  }
  bv[t] = best;
  bk[t] = kbest;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) {
      const double ov = bv[t + s];
      const int ok2 = bk[t + s];
      if (ov < bv[t] || (ov == bv[t] && ok2 < bk[t])) {
        bv[t] = ov;
        bk[t] = ok2;
      }
    }
    __syncthreads();
  }
  const int kb = bk[0];
  const double vb = bv[0];
  __syncthreads();
  double second = kInfD;
  for (int k = t; k < n_h; k += blockDim.x)
    if (k != kb) second = fmin(second, g[k]);
  bv[t] = second;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) bv[t] = fmin(bv[t], bv[t + s]);
    __syncthreads();
  }
  if (t == 0 && ok) {
    if (kb < n_h) {
      d.k_best = kb;
      d.h_best = h_dev[kb];
      d.at_edge = (kb == 0 || kb == n_h - 1) ? 1 : 0;
      d.margin = (n_h > 1) ? bv[0] - vb : 0.0;
    } else {
      d.status = kStDegenerate;  // every g(h) was NaN
    }
  }
}

// Segmented sum, block per row: *dst = sum_c src[c], fixed order.
__global__ __launch_bounds__(kThreads) void k_reduce_rows(const RowDesc* __restrict__ rows) {
  __shared__ double sh[kThreads];
  const RowDesc r = rows[blockIdx.x];
  double s = 0.0;
#pragma unroll 8
  for (int c = threadIdx.x; c < r.n; c += kThreads) s += r.src[c];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) *r.dst = s;
}

}  // namespace

// ------------------------------------------------------------------ launchers
static inline int id_blocks(int n_ids) { return (n_ids + kThreads - 1) / kThreads; }

void launch_stats(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int max_blocks, int next, int hc) {
  if (n_ids <= 0) return;
  if (max_blocks == 1) {
    k_stats_one<<<n_ids, kThreads, 0, s>>>(cols, ids, next, hc);
    return;
  }
  const dim3 grid2(max_blocks, n_ids);
  k_stats_sum<<<grid2, kThreads, 0, s>>>(cols, ids);
  k_stats_mean<<<n_ids, kThreads, 0, s>>>(cols, ids);
  k_stats_dev<<<grid2, kThreads, 0, s>>>(cols, ids);
  k_stats_final<<<n_ids, kThreads, 0, s>>>(cols, ids, next, hc);
}

void launch_plugin_step(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int step) {
  if (n_ids > 0) k_plugin_step<<<id_blocks(n_ids), kThreads, 0, s>>>(cols, ids, n_ids, step);
}

void launch_psi_scale(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids) {
  if (n_ids > 0) k_psi_scale<<<dim3(128, n_ids), kThreads, 0, s>>>(cols, ids);
}

void launch_psi_finish(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int stage, int was_f64,
                       int conditional, int next) {
  if (n_ids > 0) k_psi_finish<<<n_ids, kThreads, 0, s>>>(cols, ids, stage, was_f64, conditional, next);
}

void launch_lscv_prep(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int hc) {
  if (n_ids > 0) k_lscv_prep<<<n_ids, kThreads, 0, s>>>(cols, ids, hc);
}

void launch_lscv_finalize(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int f64) {
  if (n_ids > 0) k_lscv_finalize<<<n_ids, 1024, 0, s>>>(cols, ids, f64);
}

void launch_psi_units(hipStream_t s, int r, int f64, int conditional, int wide, const ColDesc* cols,
                      const Unit* units, int u0, int n_units) {
  if (n_units <= 0) return;
  const int t = wide ? kPsiThreads : kThreads;
#define KDE_PSI_CASE(RR)                                                                            \
  if (f64 && wide)                                                                                  \
    k_psi_wide_f64<RR><<<n_units, t, 0, s>>>(cols, units, u0, conditional);                         \
  else if (f64)                                                                                     \
    k_psi_units_f64<RR><<<n_units, t, 0, s>>>(cols, units, u0, conditional);                        \
  else if (wide)                                                                                    \
    k_psi_wide_f32<RR><<<n_units, t, 0, s>>>(cols, units, u0);                                      \
  else                                                                                              \
    k_psi_units_f32<RR><<<n_units, t, 0, s>>>(cols, units, u0);                                     \
  break
  switch (r) {
    case 8: KDE_PSI_CASE(8);
    case 6: KDE_PSI_CASE(6);
    default: KDE_PSI_CASE(4);
  }
#undef KDE_PSI_CASE
}

void launch_zero_ints(hipStream_t s, int* p, int n) {
  if (n > 0) k_zero_ints<<<(n + 255) / 256, 256, 0, s>>>(p, n);
}

// The persistent sweep's variants: (bandwidths per block, samples per LDS
// tile).  The autotuner chooses among them; (16, 512) is the default.
namespace {
template <int HC, int TJ>
int queue_blocks_of() {
  int dev = 0, per_cu = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_lscv_units_f32_queue<HC, TJ>, kThreads, 0) !=
          hipSuccess ||
      per_cu < 1)
    return 0;
  return per_cu * prop.multiProcessorCount;
}
}  // namespace

bool lscv_queue_variant(int hc, int tj) {
  return (tj == 512 && (hc == 8 || hc == 16 || hc == 32)) || (hc == 16 && (tj == 256 || tj == 1024));
}

int lscv_queue_blocks(int hc, int tj) {
  if (tj == 256) return queue_blocks_of<16, 256>();
  if (tj == 1024) return queue_blocks_of<16, 1024>();
  switch (hc) {
    case 8: return queue_blocks_of<8, 512>();
    case 32: return queue_blocks_of<32, 512>();
    default: return queue_blocks_of<16, 512>();
  }
}

void launch_lscv_units_queue(hipStream_t s, int hc, int tj, const ColDesc* cols, const Unit* units, int n_units,
                             const int* group_begin, int* next, int blocks) {
  if (n_units <= 0) return;
  blocks = max(1, min(blocks, n_units));
  if (tj == 256) {
    k_lscv_units_f32_queue<16, 256><<<blocks, kThreads, 0, s>>>(cols, units, group_begin, next);
  } else if (tj == 1024) {
    k_lscv_units_f32_queue<16, 1024><<<blocks, kThreads, 0, s>>>(cols, units, group_begin, next);
  } else {
    switch (hc) {
      case 8: k_lscv_units_f32_queue<8, 512><<<blocks, kThreads, 0, s>>>(cols, units, group_begin, next); break;
      case 32: k_lscv_units_f32_queue<32, 512><<<blocks, kThreads, 0, s>>>(cols, units, group_begin, next); break;
      default: k_lscv_units_f32_queue<16, 512><<<blocks, kThreads, 0, s>>>(cols, units, group_begin, next); break;
    }
  }
}

void launch_lscv_units(hipStream_t s, int hc, int f64, int mfma, int prune, const ColDesc* cols, const Unit* units,
                       int u0, int n_units) {
  if (n_units <= 0) return;
  if (prune && !f64) {
    switch (hc) {
      case 8: k_lscv_units_prune<8><<<n_units, kThreads, 0, s>>>(cols, units, u0, kPruneEps); break;
      case 32: k_lscv_units_prune<32><<<n_units, kThreads, 0, s>>>(cols, units, u0, kPruneEps); break;
      default: k_lscv_units_prune<16><<<n_units, kThreads, 0, s>>>(cols, units, u0, kPruneEps); break;
    }
    return;
  }
  if (mfma && !f64 && hc == 16) {
    k_lscv_units_mfma<<<n_units, kThreads, 0, s>>>(cols, units, u0);
    return;
  }
  if (f64) {
    switch (hc) {
      case 4: k_lscv_units_f64<4><<<n_units, kThreads, 0, s>>>(cols, units, u0); break;
      default: k_lscv_units_f64<8><<<n_units, kThreads, 0, s>>>(cols, units, u0); break;
    }
  } else {
    switch (hc) {
      case 8: k_lscv_units_f32<8><<<n_units, kThreads, 0, s>>>(cols, units, u0); break;
      case 32: k_lscv_units_f32<32><<<n_units, kThreads, 0, s>>>(cols, units, u0); break;
      default: k_lscv_units_f32<16><<<n_units, kThreads, 0, s>>>(cols, units, u0); break;
    }
  }
}

void launch_lscv_ceiling(hipStream_t s, int hc, const float* x, const float* c32, int reps, double* out, int blocks) {
  if (blocks <= 0) return;
  switch (hc) {
    case 8: k_lscv_ceiling<8><<<blocks, kThreads, 0, s>>>(x, c32, reps, out); break;
    case 32: k_lscv_ceiling<32><<<blocks, kThreads, 0, s>>>(x, c32, reps, out); break;
    default: k_lscv_ceiling<16><<<blocks, kThreads, 0, s>>>(x, c32, reps, out); break;
  }
}

void launch_lscv_prune_prep(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int hc, double eps) {
  if (n_ids > 0) k_lscv_prune_prep<<<n_ids, kThreads, 0, s>>>(cols, ids, hc, eps);
}

void launch_reduce_rows(hipStream_t s, const RowDesc* rows, int n_rows) {
  if (n_rows > 0) k_reduce_rows<<<n_rows, kThreads, 0, s>>>(rows);
}

}  // namespace kde
