// kde_query.hip -- the estimate's consumers: the density at query points and
// approximate range aggregates (Section 3.2: COUNT, SUM and AVG over a range
// of a numeric column from the estimated PDF), at a bandwidth chosen by the
// selectors.
//
// Density, eq. (kde-def) with d = 1 and the Gaussian kernel:
//   f(x) = (n h)^-1 sum_i phi((x - X_i) / h).
// A block holds 256 query points, one per lane, and sweeps a piece of the
// column in 512-sample LDS tiles (broadcast reads, as in the pair kernels);
// mixed form: FP32 terms via exp2 in 64-term runs folded into a compensated
// FP32 sum, FP64 across pieces, the query point carried as an FP32 pair so
// its own rounding does not shift the estimate; FP64 form: every term in
// FP64.  Padding samples hold +inf and contribute exactly zero.
//
// Range aggregates, eq. (count) and eq. (sum) with the estimate for f: the
// Gaussian kernel integrates in closed form, so for a range [a, b]
//   Count = n int_a^b f = sum_i [Phi(beta_i) - Phi(alpha_i)],
//   Sum   = n int_a^b x f = sum_i [X_i (Phi(beta_i) - Phi(alpha_i)) + h (phi(alpha_i) - phi(beta_i))],
// alpha_i = (a - X_i)/h, beta_i = (b - X_i)/h, and AVG = Sum / Count.  The
// differences of Phi are taken between tails so that ranges far from a sample
// lose no digits; everything is FP64 (O(n) terms per range).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "kde_runtime.h"

namespace kde {

namespace {

constexpr double kLog2E = 1.4426950408889634074;
constexpr double kInvSqrt2Pi = 0.39894228040143267794;
constexpr int kRunQ = 64;  // samples per plain-FP32 run before a compensated fold

__device__ __forceinline__ void fold(float& a, float& comp, float v) {
  const float y = v - comp;
  const float t = a + y;
  comp = (t - a) - y;
  a = t;
}

__device__ __forceinline__ double block_sum_q(double v, double* sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] += sh[t + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// exp2(cf (x - X)^2) over a run of kRunQ samples
__device__ __forceinline__ float density_run(const float4* __restrict__ tile, float xq, float xl, float cf) {
  float run = 0.f;
#pragma unroll 4
  for (int k = 0; k < kRunQ / 4; ++k) {
    const float4 v = tile[k];
    const float xs[4] = {v.x, v.y, v.z, v.w};
    float e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float d = (xq - xs[u]) + xl;
      e[u] = d * d * cf;
    }
    exp2_group(e);
#pragma unroll
    for (int u = 0; u < 4; ++u) run += e[u];
    __builtin_amdgcn_sched_barrier(0);
  }
  return run;
}

// grid (query blocks, pieces); part[q * pieces + piece].  Bound: vector
// issue, 8.1 cycles for the exponential and 2.4 for each of five plain
// instructions a term; the four samples of an LDS read issue their
// exponentials together (exp2_group).  n = 1e6 x 4096 points: 695 -> 563 us
// (7.3e12 terms/s, 21.6 cycles a term).
__global__ __launch_bounds__(kThreads) void k_density_f32(const ColDesc* __restrict__ col,
                                                          const double* __restrict__ q, int m, double h, int piece_len,
                                                          int pieces, double* __restrict__ part) {
  const ColDesc c = *col;
  const float* x = c.x32;
  const int qi = blockIdx.x * kThreads + threadIdx.x;
  // the query point as an FP32 pair (hi + lo): the sample differences near it
  // are then exact to FP32 rounding of the difference, not of the point
  const double xq64 = qi < m ? q[qi] - c.st->shift : 0.0;
  const float xq = (float)xq64;
  const float xl = (float)(xq64 - (double)xq);
  const float cf = (float)(-kLog2E / (2.0 * h * h));
  const int n_pad = (c.n + kBJ - 1) / kBJ * kBJ;
  const int j0 = blockIdx.y * piece_len;
  const int j1 = min(j0 + piece_len, n_pad);
  __shared__ float4 tile[kBJ / 4];
  float a = 0.f, comp = 0.f;
  for (int t0 = j0; t0 < j1; t0 += kBJ) {
    __syncthreads();
    for (int k = threadIdx.x; k < kBJ / 4; k += kThreads) tile[k] = reinterpret_cast<const float4*>(x + t0)[k];
    __syncthreads();
    for (int r0 = 0; r0 < kBJ; r0 += kRunQ) {
      fold(a, comp, density_run(tile + (r0 >> 2), xq, xl, cf));
    }
  }
  if (qi < m) part[(int64_t)qi * pieces + blockIdx.y] = (double)a - (double)comp;
}

// The same piece of the column for 64 query points, by the sixteen waves of a
// block: a run a wave and step, whose sums one wave folds in ascending order,
// so that a point's sum is the same as from k_density_f32 bit for bit.  For
// calls of few points, where a wave that is alone on its SIMD issues an
// instruction every 5-8 cycles and walks 4096 samples by itself: a call of 64
// points over n = 1e5 samples 204 -> 80 us, 512 over 1e6 209 -> 148 us.
constexpr int kWideWaves = 16;
__global__ __launch_bounds__(64 * kWideWaves) void k_density_wide_f32(const ColDesc* __restrict__ col,
                                                                      const double* __restrict__ q, int m, double h,
                                                                      int piece_len, int pieces,
                                                                      double* __restrict__ part) {
  constexpr int kTile = kRunQ * kWideWaves;
  const ColDesc c = *col;
  const float* x = c.x32;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qi = blockIdx.x * 64 + lane;
  const double xq64 = qi < m ? q[qi] - c.st->shift : 0.0;
  const float xq = (float)xq64;
  const float xl = (float)(xq64 - (double)xq);
  const float cf = (float)(-kLog2E / (2.0 * h * h));
  const int n_pad = (c.n + kBJ - 1) / kBJ * kBJ;
  const int j0 = blockIdx.y * piece_len;
  const int j1 = min(j0 + piece_len, n_pad);
  __shared__ float4 tile[kTile / 4];
  __shared__ float sums[kWideWaves][64];
  float a = 0.f, comp = 0.f;
  for (int t0 = j0; t0 < j1; t0 += kTile) {
    // every wave has swept the tile before (the second barrier below)
    if (tid < min(kTile, j1 - t0) / 4) tile[tid] = reinterpret_cast<const float4*>(x + t0)[tid];
    __syncthreads();  // the tile stands; wave 0 has folded the runs before
    if (t0 + wave * kRunQ < j1) sums[wave][lane] = density_run(tile + wave * (kRunQ / 4), xq, xl, cf);
    __syncthreads();
    if (wave == 0) {
      const int runs = min(kWideWaves, (j1 - t0) / kRunQ);
      for (int r = 0; r < runs; ++r) fold(a, comp, sums[r][lane]);
    }
  }
  if (wave == 0 && qi < m) part[(int64_t)qi * pieces + blockIdx.y] = (double)a - (double)comp;
}

__global__ __launch_bounds__(kThreads) void k_density_f64(const ColDesc* __restrict__ col,
                                                          const double* __restrict__ q, int m, double h, int piece_len,
                                                          int pieces, double* __restrict__ part) {
  const ColDesc c = *col;
  const double* x = c.x64;
  const int qi = blockIdx.x * kThreads + threadIdx.x;
  const double xq = qi < m ? q[qi] : 0.0;
  const double cd = -1.0 / (2.0 * h * h);
  const int n_pad = (c.n + kBJ - 1) / kBJ * kBJ;
  const int j0 = blockIdx.y * piece_len;
  const int j1 = min(j0 + piece_len, n_pad);
  __shared__ double tile[kBJ];
  double s = 0.0;
  for (int t0 = j0; t0 < j1; t0 += kBJ) {
    __syncthreads();
    for (int k = threadIdx.x; k < kBJ; k += kThreads) tile[k] = x[t0 + k];
    __syncthreads();
    for (int k = 0; k < kBJ; ++k) {
      const double d = xq - tile[k];
      s += exp_cw(d * d * cd);
    }
  }
  if (qi < m) part[(int64_t)qi * pieces + blockIdx.y] = s;
}

// block per query point: fixed-order sum over pieces, then the normalisation
__global__ __launch_bounds__(kThreads) void k_density_final(const ColDesc* __restrict__ col,
                                                            const double* __restrict__ part, int pieces, double h,
                                                            double* __restrict__ out) {
  __shared__ double sh[kThreads];
  const int qi = blockIdx.x;
  double s = 0.0;
  for (int p = threadIdx.x; p < pieces; p += kThreads) s += part[(int64_t)qi * pieces + p];
  s = block_sum_q(s, sh);
  if (threadIdx.x == 0) {
    const ColDesc c = *col;
    out[qi] = c.st->status != kStInval ? s * kInvSqrt2Pi / ((double)c.n * h) : NAN;
  }
}

// ---- range aggregates
// Mills' ratio of the normal law, Q(s) / phi(s) for 0 <= s <= 40: with
// t = 1 / (s + 5), M(s) = t P(y), P a polynomial of degree 22 in y, the affine
// image of t in [-1, 1] (the change of variable of Shepherd and Laframboise,
// Math. Comp. 36, 1981, for erfc; the coefficients by interpolation at the
// Chebyshev nodes with 60 digits, within 1.3e-17 of M).  The first six are
// rounded so that phi M, whose kInvSqrt2Pi is 0.56 2^-53 too large, comes out
// within 0.25 2^-53 of Q below s = 3 and 1.2 below 10 before the evaluation's
// own rounding.
__device__ __forceinline__ double mills(double s) {
  const double d = s + 5.0;
  double t = __builtin_amdgcn_rcp(d);  // about 2^-23, then two Newton steps
  t = __builtin_fma(t, __builtin_fma(-d, t, 1.0), t);
  t = __builtin_fma(t, __builtin_fma(-d, t, 1.0), t);
  const double y = __builtin_fma(t, 11.25, -1.25);
  double p = -3.394452885748163e-11;
  p = __builtin_fma(p, y, -4.502452021699791e-10);
  p = __builtin_fma(p, y, 7.631701396447264e-10);
  p = __builtin_fma(p, y, 5.72860581930563e-09);
  p = __builtin_fma(p, y, -9.579565471143506e-09);
  p = __builtin_fma(p, y, -4.877634858372001e-08);
  p = __builtin_fma(p, y, 9.378278914340451e-08);
  p = __builtin_fma(p, y, 4.1512460669879615e-07);
  p = __builtin_fma(p, y, -7.87657151045281e-07);
  p = __builtin_fma(p, y, -4.089779496515203e-06);
  p = __builtin_fma(p, y, 4.9667589688650644e-06);
  p = __builtin_fma(p, y, 4.5895086529456005e-05);
  p = __builtin_fma(p, y, 1.0093994625680667e-05);
  p = __builtin_fma(p, y, -0.0004972185327947644);
  p = __builtin_fma(p, y, -0.0013319023014207816);
  p = __builtin_fma(p, y, 0.002236503981011224);
  p = __builtin_fma(p, y, 0.02817013837425035);
  p = __builtin_fma(p, y, 0.11640743724740872);
  p = __builtin_fma(p, y, 0.324562366817339);
  p = __builtin_fma(p, y, 0.6971421572033235);
  p = __builtin_fma(p, y, 1.2141480307763557);
  p = __builtin_fma(p, y, 1.7558051918274373);
  p = __builtin_fma(p, y, 2.129871446222046);
  return t * p;
}

// phi(z), and the tail beyond z on z's side of 0: Q(|z|), negative for z < 0
// (at |z| >= 40 both are exactly 0, infinite z included).  A z of -0 counts as
// 0, here and in evaluate's comparisons: an end of -0 at a sample of 0 gives
// it, and so does a distance that underflows.
__device__ __forceinline__ void normal_tail(double z, double& phi, double& q) {
#pragma clang fp contract(off)  // equal z give equal phi: an empty range is exactly 0
  const double s = fmin(fabs(z), 40.0);
  phi = kInvSqrt2Pi * exp_cw(-0.5 * s * s);
  q = phi * mills(s);
  if (z < 0.0) q = -q;
}

// Samples whose kernel a range [a, b] does not cut need no evaluation: with
// all of 9 h inside, Phi(beta) - Phi(alpha) rounds to 1 and the densities at
// the ends are below 1e-18; 12 h or more outside the share is below 2e-33.
constexpr double kCutIn = 9.0, kCutOut = 12.0;
// A range whose COUNT is below this times n takes every sample's share as it
// is, however small (what the cut leaves out is below 2e-33 n).
constexpr double kFullBelow = 0x1p-50;

// Lanes of a wave read from LDS what other lanes of it stored: the wave's LDS
// operations execute in program order, and this keeps the compiler to that
// order (no instruction).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// grid (ranges, pieces): one range per block.  Each wave passes its samples
// once: those inside are counted, those at an end queue up in LDS until 64 of
// them fill the wave, which then evaluates them together.  FULL: every sample
// is evaluated, for the ranges flagged in need.  Bound: FP64 issue, about 100
// instructions for an evaluated sample (two exponentials, two polynomials and
// no branch), 15 for one that is not; the form before took Phi through the
// library's erfc on three branches of phi_diff, which the lanes of a wave
// shared (600 instructions a sample).  A call of n = 1e6 x 256 ranges: 3.99
// -> 0.85 ms.  Error of a single tail Q(z), on average and in 2^-53 of it: 1.9
// for z < 1, 1.7 below 3, 4.2 below 6, 15 below 12, 65 below 25 (through erfc:
// 0.8, 3.4, 14, 53, 227, nearly all of one sign); largest error of 30 calls'
// COUNTs and SUMs in 2^-53 of the largest one, on average: 1.58 and 1.55
// before, 1.44 and 1.54 now.
template <bool FULL>
__global__ __launch_bounds__(kThreads) void k_range_f64(const ColDesc* __restrict__ col, const double* __restrict__ lo,
                                                        const double* __restrict__ hi, double h, int piece_len,
                                                        int pieces, const int* __restrict__ need,
                                                        double* __restrict__ part) {
  const int r = blockIdx.x;
  if (FULL && !need[r]) return;
  const ColDesc c = *col;
  const double a = lo[r], b = hi[r];
  const double a_out = a - kCutOut * h, b_out = b + kCutOut * h, a_in = a + kCutIn * h, b_in = b - kCutIn * h;
  const double ih = 1.0 / h;
  const bool scale = !isinf(ih);  // uniform: h so small that 1 / h overflows divides
  const int i0 = blockIdx.y * piece_len;
  const int i1 = min(c.n, i0 + piece_len);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  __shared__ double queue[kThreads / 64][128];
  double cnt = 0.0, sum = 0.0;
  int inside = 0;  // uniform: samples counted whole
  auto evaluate = [&](double x) {
#pragma clang fp contract(off)
    const double al = scale ? (a - x) * ih : (a - x) / h, be = scale ? (b - x) * ih : (b - x) / h;
    double pa, pb, qa, qb;
    normal_tail(al, pa, qa);
    normal_tail(be, pb, qb);
    // between the tails on the kernel's far side: Q(al) - Q(be) for al >= 0,
    // Q(-be) - Q(-al) for be < 0, and 1 - Q(-al) - Q(be) around the sample
    double dp = qa - qb;
    if (al < 0.0 && be >= 0.0) dp += 1.0;
    cnt += dp;
    sum += x * dp + h * (pa - pb);
  };
  int queued = 0;
  for (int k0 = i0 + wave * 64; k0 < i1; k0 += kThreads) {
    const int i = k0 + lane;
    const bool valid = i < i1;
    double x = 0.0;
    if (valid)
      x = c.raw_f64 ? reinterpret_cast<const double*>(c.raw)[i] : (double)reinterpret_cast<const float*>(c.raw)[i];
    if (FULL) {
      if (valid) evaluate(x);
      continue;
    }
    const bool in = valid && x > a_in && x < b_in;
    const bool at_end = valid && !in && x >= a_out && x <= b_out;
    inside += __popcll(__ballot(in));
    if (in) sum += x;
    const uint64_t m = __ballot(at_end);
    if (at_end) queue[wave][queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = x;
    queued += __popcll(m);
    wave_order();
    if (queued >= 64) {
      queued -= 64;
      const double xq = queue[wave][queued + lane];
      wave_order();
      evaluate(xq);
    }
  }
  if (!FULL && lane < queued) evaluate(queue[wave][lane]);
  __shared__ int whole[kThreads / 64];
  if (lane == 0) whole[wave] = inside;
  __shared__ double sh[kThreads];
  cnt = block_sum_q(cnt, sh);
  sum = block_sum_q(sum, sh);
  if (threadIdx.x == 0) {
    // the whole samples last: one rounding at their size
    part[((int64_t)r * pieces + blockIdx.y) * 2] = cnt + (double)(whole[0] + whole[1] + whole[2] + whole[3]);
    part[((int64_t)r * pieces + blockIdx.y) * 2 + 1] = sum;
  }
}

// block per range: fixed-order sums over pieces; AVG = SUM / COUNT.  full: the
// second pass, over the ranges that the first one flagged.
__global__ __launch_bounds__(kThreads) void k_range_final(const ColDesc* __restrict__ col,
                                                          const double* __restrict__ part, int pieces, int full,
                                                          int* __restrict__ need, double* __restrict__ out) {
  __shared__ double sh[kThreads];
  const int r = blockIdx.x;
  if (full && !need[r]) return;
  double cnt = 0.0, sum = 0.0;
  for (int p = threadIdx.x; p < pieces; p += kThreads) {
    cnt += part[((int64_t)r * pieces + p) * 2];
    sum += part[((int64_t)r * pieces + p) * 2 + 1];
  }
  cnt = block_sum_q(cnt, sh);
  sum = block_sum_q(sum, sh);
  if (threadIdx.x == 0) {
    const bool ok = col->st->status != kStInval;
    if (!full) need[r] = ok && !(cnt >= kFullBelow * (double)col->n);
    out[3 * r] = ok ? cnt : NAN;
    out[3 * r + 1] = ok ? sum : NAN;
    out[3 * r + 2] = ok && cnt > 0.0 ? sum / cnt : NAN;
  }
}

// pieces so that a launch has about 4096 blocks, each piece at least `least`
// samples
int pieces_for(int64_t n, int64_t other_blocks, int64_t least = 4096) {
  const int64_t want = std::max<int64_t>(1, 4096 / std::max<int64_t>(1, other_blocks));
  const int64_t most = std::max<int64_t>(1, n / least);
  return (int)std::min(want, most);
}

// 64-point blocks of sixteen waves below this many blocks of 256 points (twelve
// a CU; the chip holds eight, and a last round that is partly empty costs more
// the fewer and longer the blocks are).  n = 1e6, calls of 2000, 3000, 4096
// points (1952, 2928, 3904 blocks of 256): 372, 522, 633 us in 256-point
// blocks, 363, 497, 649 us in 64-point blocks; n = 4e5, 4096 points (1568):
// 301 and 245 us.
constexpr int kDensityWide = 3072;

}  // namespace

}  // namespace kde

namespace {

using kde::fail;

bool finite_all(const double* v, int32_t m) {
  for (int32_t k = 0; k < m; ++k)
    if (!std::isfinite(v[k])) return false;
  return true;
}

}  // namespace

extern "C" {

kde_status kde_density(kde_ctx* c, kde_column x, double h, const double* points, int32_t m, double* f_out) {
  if (!c || !points || !f_out) return KDE_E_INVAL;
  if (c->server && kde::server_running(c->server.get())) return fail(c, KDE_E_BUSY, "a server is running");
  if (!(h > 0.0) || !std::isfinite(h) || m < 1 || m > KDE_MAX_QUERIES || !finite_all(points, m))
    return fail(c, KDE_E_INVAL, "need h > 0 finite, 1 <= m <= KDE_MAX_QUERIES finite points");
  if (hipSetDevice(c->device) != hipSuccess) return fail(c, KDE_E_DEVICE, "hipSetDevice failed");
  kde_status s;
  const kde::ColDesc* dcol = nullptr;
  if ((s = kde::stage_column(c, x, &dcol))) return s;
  const bool f64 = c->prec == KDE_PREC_FP64;
  const int n = (int)x.n;
  const int qblocks = (m + kde::kThreads - 1) / kde::kThreads;
  const int n_pad = (n + kde::kBJ - 1) / kde::kBJ * kde::kBJ;
  // the FP64 sums don't depend on the cut (beyond 1e-16); the compensated FP32
  // sums do (up to 1e-8 in narrow estimates), and keep theirs
  int pieces = kde::pieces_for(n_pad, qblocks, f64 ? kde::kBJ : 4096);
  int piece_len = (n_pad + pieces - 1) / pieces;
  piece_len = (piece_len + kde::kBJ - 1) / kde::kBJ * kde::kBJ;
  pieces = (n_pad + piece_len - 1) / piece_len;
  const size_t q_bytes = 8 * (size_t)m, part_bytes = 8 * (size_t)m * pieces;
  if ((s = kde::ensure(c, c->qbuf, q_bytes + part_bytes + q_bytes + 768))) return s;
  char* base = c->qbuf.p;
  double* dq = (double*)base;
  double* dpart = (double*)(base + (q_bytes + 255) / 256 * 256);
  double* dout = (double*)((char*)dpart + (part_bytes + 255) / 256 * 256);
  KDE_HIP_TRY(c, hipMemcpyAsync(dq, points, q_bytes, hipMemcpyHostToDevice, c->stream));
  const dim3 grid(qblocks, pieces);
  if (f64)
    kde::k_density_f64<<<grid, kde::kThreads, 0, c->stream>>>(dcol, dq, m, h, piece_len, pieces, dpart);
  else if (qblocks * pieces < kde::kDensityWide)
    kde::k_density_wide_f32<<<dim3((m + 63) / 64, pieces), 64 * kde::kWideWaves, 0, c->stream>>>(
        dcol, dq, m, h, piece_len, pieces, dpart);
  else
    kde::k_density_f32<<<grid, kde::kThreads, 0, c->stream>>>(dcol, dq, m, h, piece_len, pieces, dpart);
  kde::k_density_final<<<m, kde::kThreads, 0, c->stream>>>(dcol, dpart, pieces, h, dout);
  KDE_HIP_TRY(c, hipMemcpyAsync(f_out, dout, q_bytes, hipMemcpyDeviceToHost, c->stream));
  return kde::sync_and_check(c);
}

kde_status kde_range_aggregates(kde_ctx* c, kde_column x, double h, const double* lo, const double* hi, int32_t q,
                                double* count_out, double* sum_out, double* avg_out) {
  if (!c || !lo || !hi || !count_out || !sum_out) return KDE_E_INVAL;
  if (c->server && kde::server_running(c->server.get())) return fail(c, KDE_E_BUSY, "a server is running");
  if (!(h > 0.0) || !std::isfinite(h) || q < 1 || q > KDE_MAX_QUERIES)
    return fail(c, KDE_E_INVAL, "need h > 0 finite and 1 <= q <= KDE_MAX_QUERIES");
  for (int32_t k = 0; k < q; ++k)
    if (std::isnan(lo[k]) || std::isnan(hi[k]) || !(lo[k] <= hi[k]))
      return fail(c, KDE_E_INVAL, "every range needs lo <= hi (infinite ends allowed)");
  if (hipSetDevice(c->device) != hipSuccess) return fail(c, KDE_E_DEVICE, "hipSetDevice failed");
  kde_status s;
  const kde::ColDesc* dcol = nullptr;
  if ((s = kde::stage_column(c, x, &dcol))) return s;
  const int n = (int)x.n;
  int pieces = kde::pieces_for(n, q);
  const int piece_len = (n + pieces - 1) / pieces;
  pieces = (n + piece_len - 1) / piece_len;
  const size_t r_bytes = 8 * (size_t)q, part_bytes = 16 * (size_t)q * pieces, out_bytes = 24 * (size_t)q;
  if ((s = kde::ensure(c, c->qbuf, 2 * r_bytes + part_bytes + out_bytes + 4 * (size_t)q + 1280))) return s;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  char* base = c->qbuf.p;
  double* dlo = (double*)base;
  double* dhi = (double*)(base + al(r_bytes));
  double* dpart = (double*)(base + 2 * al(r_bytes));
  double* dout = (double*)(base + 2 * al(r_bytes) + al(part_bytes));
  int* dneed = (int*)((char*)dout + al(out_bytes));
  KDE_HIP_TRY(c, hipMemcpyAsync(dlo, lo, r_bytes, hipMemcpyHostToDevice, c->stream));
  KDE_HIP_TRY(c, hipMemcpyAsync(dhi, hi, r_bytes, hipMemcpyHostToDevice, c->stream));
  const dim3 grid(q, pieces);
  kde::k_range_f64<false>
      <<<grid, kde::kThreads, 0, c->stream>>>(dcol, dlo, dhi, h, piece_len, pieces, dneed, dpart);
  kde::k_range_final<<<q, kde::kThreads, 0, c->stream>>>(dcol, dpart, pieces, 0, dneed, dout);
  kde::k_range_f64<true><<<grid, kde::kThreads, 0, c->stream>>>(dcol, dlo, dhi, h, piece_len, pieces, dneed, dpart);
  kde::k_range_final<<<q, kde::kThreads, 0, c->stream>>>(dcol, dpart, pieces, 1, dneed, dout);
  std::vector<double> out(3 * (size_t)q);
  KDE_HIP_TRY(c, hipMemcpyAsync(out.data(), dout, out_bytes, hipMemcpyDeviceToHost, c->stream));
  if ((s = kde::sync_and_check(c))) return s;
  for (int32_t k = 0; k < q; ++k) {
    count_out[k] = out[3 * (size_t)k];
    sum_out[k] = out[3 * (size_t)k + 1];
    if (avg_out) avg_out[k] = out[3 * (size_t)k + 2];
  }
  return KDE_OK;
}

}  // extern "C"
