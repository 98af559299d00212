// kde_internal.h -- types shared by the kernels and the host runtime of the
// bandwidth-selection library.  Not part of the public ABI (see kde_bw.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kde {

// Threads per block of every pair kernel: four 64-wide waves.  Each block
// owns one "row" of kBI consecutive samples i (one per lane).
constexpr int kThreads = 256;
constexpr int kBI = kThreads;
// Threads per block of the psi kernels of smaller columns: 16 waves share the
// runs of 64 samples i.  A work item's row of kBI samples is kPsiGroups such
// units.
constexpr int kPsiThreads = 1024;
constexpr int kPsiGroups = kBI / 64;
// j-tile staged in LDS per step; item j-ranges are whole multiples of it.
constexpr int kBJ = 512;
// Every column is padded with +inf up to at least n + kPad so that every
// tile read stays in bounds and padded j contribute exactly zero.
constexpr int kPad = kBJ + kBI;
// Blocks per column of the moment passes (a column of n samples uses
// min(kStatBlocks, ceil(n / 2048)) of them).
constexpr int kStatBlocks = 1024;

// Tile pruning: the skipped share of every pair sum is below this fraction
// of the sum (2^-34).
constexpr double kPruneEps = 5.820766091346741e-11;

// Status values written by device code (same numbers as kde_status).
constexpr int kStOk = 0;
constexpr int kStInval = 1;
constexpr int kStDegenerate = 2;

// Grid kinds of an LSCV request (match kde_grid_kind in kde_bw.h).
constexpr int kGridExplicit = 0;
constexpr int kGridPaper = 1;    // linear over sigma * [h0/4, 4 h0]
constexpr int kGridLogRot = 2;   // log-spaced over h_rot * [lo, hi]

// e^x in FP64 for the pair loops (arguments <= 0: x = -D^2 c), by Cody and
// Waite's argument reduction: k = nearest integer to x / ln 2, read from the
// low bits of x / ln 2 + 1.5 2^52, r = x - k ln 2 with ln 2 split into a head
// of 29 significant bits (k * head is exact for |k| < 2^24, so x - k * head is
// exact) and a tail, |r| <= ln(2) / 2; then 1 + r + r^2 / 2 + r^3 q(r) and the
// scaling by 2^k.  q is the polynomial of degree 9 of least maximal relative
// error in e^r there (Lawson's reweighted least squares in 60 digits; 5.9e-20,
// where the Taylor series to r^13 leaves 4.1e-18).  18 instructions; with the
// series, a rounding and a conversion of k it was 20, at 4.3 cycles a wave
// each.  Error over [-708, 0], in 2^-53: at most 1.23, 0.369 on average (the
// series: 1.25 and 0.370); a q of degree 8 with a free r^2 term reached 1.30.
// Arguments below -1100 (and -inf) are raised to -1100, which underflows to
// exactly 0; no NaN arrives here (samples are finite, and masked pairs carry
// -inf).
__device__ __forceinline__ double exp_cw(double x) {
  constexpr double kInvLn2 = 1.4426950408889634;
  constexpr double kLn2Head = 0x1.62e42ffp-1;         // ln 2 rounded to 29 bits
  constexpr double kLn2Tail = -4.2009150726810846e-11;  // ln 2 - head
  constexpr double kRound = 0x1.8p52;
  x = fmax(x, -1100.0);
  const double t = __builtin_fma(x, kInvLn2, kRound);
  const double k = t - kRound;
  double r = __builtin_fma(-k, kLn2Head, x);
  r = __builtin_fma(-k, kLn2Tail, r);
  double p = 2.0838694141142642e-09;
  p = __builtin_fma(p, r, 2.5111246787424845e-08);
  p = __builtin_fma(p, r, 2.755752550233924e-07);
  p = __builtin_fma(p, r, 2.7557237450030694e-06);
  p = __builtin_fma(p, r, 2.4801587026265436e-05);
  p = __builtin_fma(p, r, 0.00019841269893349788);
  p = __builtin_fma(p, r, 0.001388888888903298);
  p = __builtin_fma(p, r, 0.008333333333318522);
  p = __builtin_fma(p, r, 0.041666666666666415);
  p = __builtin_fma(p, r, 0.1666666666666668);
  p = __builtin_fma(p, r, 0.5);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  return ldexp(p, (int)(uint32_t)__builtin_bit_cast(uint64_t, t));
}

// ---- sums over the 64 lanes of a wave, all lanes active, in vector registers
// (row permutes and lane swaps; no LDS traffic).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Each row of 16 lanes: every lane gets its row's sum.
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_f64<0xB1>(v);   // lane ^ 1
  v += dpp_f64<0x4E>(v);   // lane ^ 2
  v += dpp_f64<0x141>(v);  // the other half of 8
  v += dpp_f64<0x140>(v);  // the other half of 16
  return v;
}

// a + b with the upper half of a exchanged for the lower half of b: lanes
// 0 - 31 get a[l] + a[l + 32], lanes 32 - 63 get b[l - 32] + b[l].
__device__ __forceinline__ double swap32_add(double a, double b) {
  const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
  return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
         __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

// The same between neighbouring rows of 16: rows 0 and 2 get a's two rows
// added, rows 1 and 3 b's.
__device__ __forceinline__ double swap16_add(double a, double b) {
  const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
  return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
         __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

// Sums of N values over the wave's lanes into out[0 .. N) (N a multiple of
// 4): two exchange steps leave N / 4 values a lane, row r of 16 lanes holding
// values r N / 4 and up, and the rows are summed in place.  3 N / 2 exchanges
// and sums plus 3 N row steps against 18 N LDS permutes and sums of a full
// butterfly per value; the order of every sum does not depend on N.
template <int N>
__device__ __forceinline__ void wave_sums(const double (&v)[N], double* out, int lane) {
  double h[N / 2];
#pragma unroll
  for (int k = 0; k < N / 2; ++k) h[k] = swap32_add(v[k], v[k + N / 2]);
#pragma unroll
  for (int k = 0; k < N / 4; ++k) {
    const double s = row16_sum(swap16_add(h[k], h[k + N / 4]));
    if ((lane & 15) == 0) out[(lane >> 4) * (N / 4) + k] = s;
  }
}

// Two values: lane 0 gets the sum of a, lane 32 the sum of b.
__device__ __forceinline__ double wave_sum2(double a, double b) {
  const double s = swap32_add(a, b);
  return row16_sum(swap16_add(s, s));
}

// Exponentials issued together in the FP32 pair loops (2: 1% slower in the
// LSCV sweep, 8: 1% slower).
constexpr int kExpGroup = 4;

// e[k] = exp2(e[k]) for a group of arguments, issued back to back at raised
// wave priority.  The empty asm statements pin the order: the arguments are
// complete before the priority rises, the exponentials lie between the two
// priority changes, and nothing of the caller's moves in.
template <int N>
__device__ __forceinline__ void exp2_group(float (&e)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) asm volatile("" : "+v"(e[k]));
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    e[k] = __builtin_amdgcn_exp2f(e[k]);
    asm volatile("" : "+v"(e[k]));
  }
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
}

// Device-resident state of one column of a job.  All scalar steps of the
// method run on the device and read/write this struct, so a whole job is a
// chain of kernels on one stream with one copy back at the end.
struct DevState {
  int status;       // column status (invalid sample, zero spread)
  int pstatus;      // plug-in status (a pilot or final radicand not positive)
  int active;       // the current plug-in stage applies to this column
  int need_f64;     // mixed precision: current plug-in stage is re-run in FP64
  int k_best;
  int at_edge;
  int prec_used[3];
  int stages;       // plug-in stages (2 or 3); 0 when the column has no plug-in
  int pad0;
  double n;
  double shift;     // subtracted from float64 samples before rounding to float32
  double mean, var, sigma, h_rot;
  double g[3], psi[3], kappa[3];
  double h_plugin;
  double h_best, margin;
  double fp64_kappa;  // kappa threshold for the FP64 re-run (0 = never)
  float psi_scale;  // FP32 1/g of the current psi pass (its samples are x32 * psi_scale)
  int psi_fast;     // the scaled copy's range keeps every Hermite value finite (no clamp needed)
  double cd[2];     // FP64 pair coefficients: 1/g^2, -1/(2 g^2)
  float xmin, xmax; // range of the FP32 working copy
  double pruned_evals;  // LSCV pair-term evaluations skipped by tile pruning (exact count)
};

// One column of a job: where its data, coefficients, partial sums and state
// live (absolute device addresses, so resident columns of a server and the
// packed columns of a batch are described the same way).
struct ColDesc {
  const void* raw;      // input samples, float32 or float64
  float* x32;           // padded FP32 working copy [n + kPad]
  float* y32;           // psi pass of a large column: the working copy times 1/g of the stage [n + kPad] (may be null)
  double* x64;          // padded FP64 working copy [n + kPad] (may be null)
  double* stat;         // moment partials [kStatBlocks]
  float* stat_mm;       // minimum and maximum partials of the FP32 working copy [2][kStatBlocks]
  int* stat_nf;         // non-finite counts [kStatBlocks]
  double* psi_part;     // psi partials [2][n_items_psi]
  double* psi_sums;     // [2]
  const double* h_in;   // explicit grid [n_h]
  double* h;            // grid used [n_chunks * HC]
  float* c32;           // FP32 exponent coefficients [n_chunks * HC]
  double* c64;          // FP64 exponent coefficients [n_chunks * HC]
  double* part;         // LSCV partials [2 n_h][n_items], row = 2 h + {0, 1}
  double* sums;         // LSCV pair sums [2 n_h]
  double* g;            // g(h) [n_h]
  double* gs;           // gscale(h) [n_h]
  double* near_sums;    // tile pruning: pair sums of each row's first j-tile [2 n_h] (lower bounds)
  float* d2cut;         // tile pruning: squared distance beyond which a tile is skipped, per chunk
  DevState* st;
  int n;
  int raw_f64;
  int n_h;              // LSCV grid points (0: no LSCV for this column)
  int n_chunks;         // ceil(n_h / HC)
  int n_items;          // LSCV partial-sum slots a bandwidth (work items x pieces)
  int n_items_psi;      // psi partial-sum slots (work items x psi_groups)
  int grid_kind;        // kGridExplicit / kGridPaper / kGridLogRot
  int lscv_piece;       // samples j an LSCV partial-sum slot, where items are cut into pieces (0: a unit has one slot)
  double grid_lo, grid_hi;
};

// One block of a pair kernel: the samples i in [row*kBI, row*kBI + kBI) (psi
// with chunk 1: [row*64, row*64 + 64)) of column `col` against j in
// [j_begin, j_end) (a multiple of 64 long; a column's last unit may run past n
// into the +inf padding).  `item` is the (first) partial-sum slot within the
// column (its work item, times the slots of an item, plus the unit's place in
// it), `chunk` the bandwidth chunk (LSCV) or the psi geometry (0: rows of kBI
// samples, 1: of 64).
struct Unit {
  int col, row, j_begin, j_end, item, chunk;
};

// One row of a segmented reduction: *dst = sum of src[0 .. n).
struct RowDesc {
  const double* src;
  double* dst;
  int n;
  int pad0;
};

// ---- launchers (kde_kernels.hip); all asynchronous on `s` ----
// Column-level launches act on the columns cols[ids[0 .. n_ids)].
// A step of the plug-in rule, by one thread of a column: 0, 1, 2: the pilot
// bandwidth of that stage; kStepFinal: the bandwidth from psi_4; -1: none.
constexpr int kStepFinal = 3;
// Moments and normal-reference bandwidth, then the step `next` and, with
// hc > 0, the bandwidth grid (launch_lscv_prep) of the same columns.
void launch_stats(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int max_blocks, int next, int hc);
void launch_plugin_step(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int step);
// Mixed form, large columns: the scaled copy y32 = x32 / g of every active column.
void launch_psi_scale(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids);
// Sums of the units' partials, the stage's functional, then the step `next`.
void launch_psi_finish(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int stage, int was_f64,
                       int conditional, int next);
void launch_lscv_prep(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int hc);
void launch_lscv_finalize(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int f64);
// Pair kernels act on units[u0 .. u0 + n_units).  wide: units of 64 samples i.
void launch_psi_units(hipStream_t s, int r, int f64, int conditional, int wide, const ColDesc* cols,
                      const Unit* units, int u0, int n_units);
// mfma: use the matrix-core variant (FP32, 16 bandwidths per unit only).
// Tile pruning: per column, the cut distance of every bandwidth chunk from
// the near-tile sums (relative bound eps on every skipped share).
void launch_lscv_prune_prep(hipStream_t s, const ColDesc* cols, const int* ids, int n_ids, int hc, double eps);
// The sweep's inner loop over one LDS tile (x: kBJ samples, c32: hc
// coefficients), reps times per block; out: blocks x 4 doubles.
void launch_lscv_ceiling(hipStream_t s, int hc, const float* x, const float* c32, int reps, double* out, int blocks);
void launch_lscv_units(hipStream_t s, int hc, int f64, int mfma, int prune, const ColDesc* cols, const Unit* units,
                       int u0, int n_units);
void launch_reduce_rows(hipStream_t s, const RowDesc* rows, int n_rows);
// Persistent form of the dense FP32 LSCV sweep: `blocks` blocks take the
// n_units units from kQueueGroups groups, group g being units
// [group_begin[g], group_begin[g + 1]) (device array of kQueueGroups + 1
// ints, group_begin[kQueueGroups] = n_units) with device counter next[g]
// (kQueueGroups ints, all 0 at launch: clear them with launch_zero_ints in
// the same stream).  Variants (hc bandwidths per block, tj samples per LDS
// tile): (8, 512), (16, 256), (16, 512), (16, 1024), (32, 512);
// lscv_queue_variant says whether one exists.  lscv_queue_blocks: the blocks
// the current device holds at once for a variant (0 on failure).
constexpr int kQueueGroups = 8;
void launch_zero_ints(hipStream_t s, int* p, int n);
bool lscv_queue_variant(int hc, int tj);
int lscv_queue_blocks(int hc, int tj);
void launch_lscv_units_queue(hipStream_t s, int hc, int tj, const ColDesc* cols, const Unit* units, int n_units,
                             const int* group_begin, int* next, int blocks);

// ---- ascending sort of FP32 keys (kde_sort.hip): temporary bytes for
// `count` keys (0 on failure), and the sort itself.
size_t sort_temp_bytes(int count);
hipError_t sort_keys(void* tmp, size_t tmp_bytes, const float* in, float* out, int count, hipStream_t s);

}  // namespace kde
