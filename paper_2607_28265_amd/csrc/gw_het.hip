// Heterodyned (relative-binning) likelihood, Sec. III.D.
//
// Set-up (once per reference parameters theta0): bin edges of equal maximum
// phase change on the host, then on the device the reference phase at the
// edges and the per-detector summary data A0, A1 (data x reference) and
// B0, B1 (reference norm) per bin, by segmented sums over the fine grid with a
// fixed-order workgroup reduction.
//
// Evaluation: one lane per proposal, edge records wave-uniform (scalar loads).
// For TaylorF2 without a cut-off the ratio r_i = h_i / h0_i at an edge is
// (A P_i / A0 P0_i) exp(-2 pi i (Phi_i - Phi0_i)); the complex prefactor is
// pulled out of the bin sums, so per edge a lane evaluates the FP64 phase
// difference per detector, one phasor each, and the linear-in-bin contraction
// with the summary data.  Work arrives as a device-resident list of
// (row offset, count) sub-batches; a persistent grid of waves walks 64-row
// tiles of that list, so one launch (and one captured hipGraph) serves any
// sub-batch layout.  The distance marginal is evaluated inside the same wave.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <vector>

#include "gw_ctx.h"
#include "gw_hetplan.h"
#include "gw_tgrid.h"

// Device-resident arguments of the work-list kernels; a one-thread kernel
// writes them before each launch so that a captured graph can be replayed
// with new buffers.
struct HetArgs {
  const double* theta;
  const int64_t* subs;  // (row offset, count) pairs
  double* logl;
  double* coef;         // per-row coefficients [C_NCOEF][ld]
  double* zbuf;         // per-row (|Z_1|, <h|h>_1) [2][ld] for the distance marginal
  double* part;         // per-row partial sums [edge chunk][3 n_det][ld]
  int64_t n_rows;
  int64_t ld;
  int32_t n_sub;
  int32_t pad;
  double* zcplx;        // or NULL: per-row (Re Z, Im Z, <h|h>) [3][ld] for post-hoc reconstruction
};

struct gw_het_state {
  int n_bins = 0;
  int n_edges = 0;
  int rs = 0;                    // record stride (doubles)
  double* rec = nullptr;         // [n_edges][rs]
  std::vector<double> f_edges;   // host copy
  std::vector<double> theta0;
  double ap0_inv_re[gw::kMaxDet] = {0};
  double ap0_inv_im[gw::kMaxDet] = {0};
  double hh0[gw::kMaxDet] = {0};  // sum_b B0_b / 2 per detector (unit-phasor <h|h> constant)
  // work-list machinery
  HetArgs* args = nullptr;       // device
  int64_t* tile_pre = nullptr;   // device [max_sub + 1]
  int64_t* subs_single = nullptr;  // device [2]
  int max_sub = 0;
  // launch shape of the evaluation kernel
  int wpb = 4;                   // waves per workgroup
  int grid = 0;                  // workgroups (0 = heuristic)
  int ech = 0;                   // edge chunks (0 = heuristic)
  int64_t n_rows_last = 0;       // rows of the batch being enqueued (selects the distance form)
  // a caller that evaluates the same single batch (theta, rows, logl) many
  // times in a row writes the argument block once (het_pin_args); meanwhile
  // matching calls launch no k_set_args
  bool args_pinned = false;
  const double* pin_theta = nullptr;
  const double* pin_logl = nullptr;
  int64_t pin_rows = 0;
  // time marginal: row-independent tables for the current grid (built on
  // first use): per edge the kTgW grid weights and the powers sigma_e^m of its
  // bin width about the widths' centre (m < tm_mh), and the moment kernel's
  // chunks (gw_hetplan.h)
  double* tm_tab = nullptr;      // [n_edges][kTgW + tm_mh]
  // the cover's points (gw_tgrid.h), the cell of each edge [n_edges] (tm_cell),
  // the chunks' first edge [nch + 1], first cell, end cell and first point
  // [nch] each, the cover's shifts
  int32_t* tm_idx = nullptr;
  const int32_t* tm_cell = nullptr;
  TgCover tm_cov;
  int tm_blk = 0, tm_nblk = 0, tm_mh = 0, tm_nch = 0, tm_nch_req = -1, tm_L = 0, tm_jmax = -1;
  int tm_npts = 0;               // grid points of a row's chunks
  double tm_hw = 0.0;            // half-range of the bin widths (fine bins)
  int64_t tm_c2 = 0;             // smallest + largest bin width (fine bins)
};

struct GraphKey {
  int marg, prec, wpb, grid, n_ech, sliced;
  bool operator<(const GraphKey& o) const {
    return std::tie(marg, prec, wpb, grid, n_ech, sliced) < std::tie(o.marg, o.prec, o.wpb, o.grid, o.n_ech, o.sliced);
  }
};

struct gw_graph_cache {
  std::map<GraphKey, hipGraphExec_t> exec;
  std::map<GraphKey, hipGraph_t> graph;
  hipStream_t cap_stream = nullptr;
  double last_instantiate_ms = 0.0;
};

namespace gw {

constexpr int kMaxSub = 1 << 16;

// Record layout of one edge e (bin e-1 data rides along with edge e).
__host__ __device__ constexpr int het_rs(int nd) { return 6 + 7 * nd; }
enum HetRec { H_X = 0, H_X2 = 1, H_XM5 = 2, H_LNF = 3, H_F = 4, H_PHI0 = 5 };  // then f dtau0_i (i >= 1)
__host__ __device__ constexpr int het_bin_off(int nd) { return 5 + nd; }      // inv width, then 6 per det
// The 6 per-detector slots of edge e first receive the summary data of bin e
// (between edges e-1 and e): A0 (re, im), A1 (re, im), B0, 2 B1.  The set-up
// then rewrites them as per-edge weights of the summed-by-parts bin sums
// (see k_het): C_e = R_e + L_{e+1} (re, im), R_e (re, im), B0_e / 2, 0, with
// R_e = A0_e / 2 + A1_e / w_e and L_e = A0_e / 2 - A1_e / w_e (w_e the width
// of bin e; R_0 = L_{n+1} = 0, B0_0 = 0).

// ---------------------------------------------------------------------------
// Set-up kernels

__global__ void k_het_edges(const double* __restrict__ bins, int bin_rs, const int64_t* __restrict__ edge_idx,
                            int n_edges, int nd, const double* __restrict__ coef0, TrigConsts T, int64_t k0,
                            double df, double* __restrict__ rec) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_edges) return;
  const int rs = het_rs(nd);
  const int64_t k = edge_idx[e];
  const double* b = bins + k * bin_rs;
  PhaseCoef c;
  c.a0 = coef0[C_A0]; c.a2 = coef0[C_A2]; c.a3 = coef0[C_A3]; c.a4 = coef0[C_A4];
  c.a5 = coef0[C_A5]; c.a6 = coef0[C_A6]; c.a7 = coef0[C_A7]; c.a8 = coef0[C_A8];
  c.a10 = coef0[C_A10]; c.a12 = coef0[C_A12]; c.b5 = coef0[C_B5]; c.b6 = coef0[C_B6];
  const double f = (double)(k0 + k) * df;
  double* r = rec + (int64_t)e * rs;
  r[H_X] = b[0];
  r[H_X2] = b[1];
  r[H_XM5] = b[2];
  r[H_LNF] = b[3];
  r[H_F] = f;
  r[H_PHI0] = phase_cycles(c, b[0], b[1], b[2], b[3]);
  for (int i = 1; i < nd; ++i) r[H_PHI0 + i] = f * coef0[C_DT1 + i - 1];
  const int bo = het_bin_off(nd);
  if (e > 0) {
    const double fl = (double)(k0 + edge_idx[e - 1]) * df;
    r[bo] = 1.0 / (f - fl);
  } else {
    for (int j = bo; j < rs; ++j) r[j] = 0.0;
  }
  (void)T;
}

// One workgroup per (bin, detector): segmented sums over the fine bins of the
// bin with a fixed-order LDS tree.
__global__ void __launch_bounds__(256) k_het_summary(const double* __restrict__ bins, int bin_rs,
                                                     const double* __restrict__ hw, int64_t n_freq,
                                                     const int64_t* __restrict__ edge_idx, int n_bins,
                                                     const double* __restrict__ coef0, TrigConsts T, int64_t k0,
                                                     double df, double* __restrict__ rec, int nd) {
  const int b = blockIdx.x;
  const int i = blockIdx.y;
  const int64_t lo = edge_idx[b];
  const int64_t hi = edge_idx[b + 1];
  const int64_t stop = (b == n_bins - 1) ? hi + 1 : hi;
  const double fc = 0.5 * ((double)(k0 + lo) + (double)(k0 + hi)) * df;
  PhaseCoef c;
  c.a0 = coef0[C_A0]; c.a2 = coef0[C_A2]; c.a3 = coef0[C_A3]; c.a4 = coef0[C_A4];
  c.a5 = coef0[C_A5]; c.a6 = coef0[C_A6]; c.a7 = coef0[C_A7]; c.a8 = coef0[C_A8];
  c.a10 = coef0[C_A10]; c.a12 = coef0[C_A12]; c.b5 = coef0[C_B5]; c.b6 = coef0[C_B6];
  const double dt = i == 0 ? 0.0 : coef0[C_DT1 + i - 1];
  const double apr = coef0[C_APRE + i], api = coef0[C_APIM + i];
  const double ap2 = apr * apr + api * api;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int64_t k = lo + threadIdx.x; k < stop; k += blockDim.x) {
    const double* r = bins + k * bin_rs;
    const double f = (double)(k0 + k) * df;
    const double ph = phase_cycles(c, r[0], r[1], r[2], r[3]) + f * dt;
    double s, co;
    sincos_cycles(ph, T, &s, &co);
    // 4 df d* h0 / S = u_ik (A P0_i) exp(-2 pi i phi)
    const double ur = r[4 + 2 * i], ui = r[5 + 2 * i];
    const double gr = apr * co + api * s, gi = api * co - apr * s;
    const double tr = ur * gr - ui * gi, ti = ur * gi + ui * gr;
    const double w = ap2 * hw[(int64_t)i * n_freq + k];
    const double dfc = f - fc;
    acc[0] += tr;
    acc[1] += ti;
    acc[2] += tr * dfc;
    acc[3] += ti * dfc;
    acc[4] += w;
    acc[5] += w * dfc;
  }
  __shared__ double red[6][256];
  for (int j = 0; j < 6; ++j) red[j][threadIdx.x] = acc[j];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o)
      for (int j = 0; j < 6; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* r = rec + (int64_t)(b + 1) * het_rs(nd) + het_bin_off(nd) + 1 + 6 * i;
    r[0] = red[0][0];
    r[1] = red[1][0];
    r[2] = red[2][0];
    r[3] = red[3][0];
    r[4] = red[4][0];
    r[5] = 2.0 * red[5][0];  // 2 B1
  }
}

// ---------------------------------------------------------------------------
// Work-list kernels

// Writes the argument block and the prefix sums of 64-row tiles per
// sub-batch (pre[s] = tiles before sub-batch s, pre[n_sub] = all tiles) in one
// launch of 256 threads.  ``subs`` is read from the device; a single batch
// (subs_single != NULL) is described by (0, single_n) without reading it back.
__global__ void __launch_bounds__(256) k_set_args(HetArgs* a, const double* theta, const int64_t* subs, double* logl,
                                                  double* coef, double* zbuf, double* part, int64_t n_rows,
                                                  int32_t n_sub, int64_t* subs_single, int64_t single_n,
                                                  int64_t* __restrict__ pre, double* zcplx) {
  if (threadIdx.x == 0) {
    a->zcplx = zcplx;
    a->theta = theta;
    a->subs = subs;
    a->logl = logl;
    a->coef = coef;
    a->zbuf = zbuf;
    a->part = part;
    a->n_rows = n_rows;
    a->ld = n_rows;
    a->n_sub = n_sub;
    a->pad = 0;
    if (subs_single) {
      subs_single[0] = 0;
      subs_single[1] = single_n;
    }
  }
  if (subs_single) {
    if (threadIdx.x == 0) {
      pre[0] = 0;
      pre[1] = n_rows > 0 ? (n_rows + 63) / 64 : 0;
    }
    return;
  }
  __shared__ int64_t acc[256];
  const int per = (n_sub + 255) / 256;
  const int s0 = threadIdx.x * per;
  const int s1 = min(s0 + per, n_sub);
  int64_t sum = 0;
  for (int q = s0; q < s1; ++q) {
    int64_t cnt = subs[2 * q + 1];
    const int64_t off = subs[2 * q];
    if (off < 0 || off >= n_rows || cnt <= 0) cnt = 0;
    else if (cnt > n_rows - off) cnt = n_rows - off;
    sum += (cnt + 63) / 64;
  }
  acc[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int j = 0; j < 256; ++j) {
      const int64_t v = acc[j];
      acc[j] = run;
      run += v;
    }
    pre[n_sub] = run;
  }
  __syncthreads();
  int64_t run = acc[threadIdx.x];
  for (int q = s0; q < s1; ++q) {
    pre[q] = run;
    int64_t cnt = subs[2 * q + 1];
    const int64_t off = subs[2 * q];
    if (off < 0 || off >= n_rows || cnt <= 0) cnt = 0;
    else if (cnt > n_rows - off) cnt = n_rows - off;
    run += (cnt + 63) / 64;
  }
}

// Tile t of the work list -> (first row, one-past-last row); returns false
// for an empty tile.
__device__ inline bool tile_rows(const HetArgs* __restrict__ ab, const int64_t* __restrict__ pre, int64_t t,
                                 int64_t* row0, int64_t* row_end) {
  int lo = 0, hi = ab->n_sub;  // invariant pre[lo] <= t < pre[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= t) lo = mid;
    else hi = mid;
  }
  const int64_t off = ab->subs[2 * lo];
  int64_t cnt = ab->subs[2 * lo + 1];
  if (cnt > ab->n_rows - off) cnt = ab->n_rows - off;
  *row0 = off + (t - pre[lo]) * 64;
  *row_end = off + cnt;
  return *row0 < *row_end;
}

// Per-row prologue over the work list (same tiles as the evaluation kernel): a
// workgroup per 64-row tile, wave 0 taking the phase half of the prologue and
// wave 1 the sky half (see k_prologue).
__global__ void __launch_bounds__(128) k_het_prologue(const HetArgs* __restrict__ ab,
                                                      const int64_t* __restrict__ pre, int marg, Geom geom) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t total = pre[ab->n_sub];
  const int64_t ld = ab->ld;
  for (int64_t t = blockIdx.x; t < total; t += gridDim.x) {
    int64_t row0, row_end;
    if (!tile_rows(ab, pre, t, &row0, &row_end)) continue;
    const int64_t p = row0 + lane;
    if (p >= row_end) continue;
    const Row row = load_row(ab->theta + p * 13, marg);
    if (wave == 0) prologue_phase(row, marg, ab->coef + p, ld);
    else prologue_sky(row, marg, geom, ab->coef + p, ld);
  }
}

struct HetConst {
  double ap0_inv_re[kMaxDet];
  double ap0_inv_im[kMaxDet];
  double hh0[kMaxDet];
  double dd;
};

// exp(-2 pi i r), FP64, from tab [256] = (cos, sin)(2 pi k / 256) in LDS:
// |a| <= pi / 256 about the nearest point, cos a - 1 and sin a by their Taylor
// polynomials (first dropped terms 1.3e-20 and 8e-18).  The sum r + 1.5 2^44
// rounds r to 1/256 and its low bits are the table index: it holds for |r| < 2^43
// cycles (a row far from the reference, or hours away in t_c; a conversion to 32
// bits would saturate from 2^23 on).  17 vector operations and a gather against 31
// of sincos_cycles; k_het has LDS time to spare.  20,011 rows of 5000 bins take 394
// us and 6481 rows of 726 bins 54.6, against 408 and 56.6 with 256 r rounded and
// converted.
__device__ inline void het_phasor_tab(double r, const double2* __restrict__ tab, double* gr, double* gi) {
  constexpr double kRound = 26388279066624.0;  // 1.5 2^44: the sum rounds to 1/256
  const double m = r + kRound;
  const double a = (r - (m - kRound)) * kTwoPi;
  const double2 t = tab[__double2loint(m) & 255];
  const double a2 = a * a;
  const double sn = fma(a * a2, fma(a2, 1.0 / 120.0, -1.0 / 6.0), a);
  const double cm = a2 * fma(a2, fma(a2, -1.0 / 720.0, 1.0 / 24.0), -0.5);
  *gr = fma(t.x, cm, fma(-t.y, sn, t.x));
  *gi = -fma(t.y, cm, fma(t.x, sn, t.y));
}

template <int PREC>
__device__ inline void het_phasor(double r, const TrigConsts& T, double* gr, double* gi) {
  if (PREC == 0) {
    double s, c;
    sincos_cycles(r, T, &s, &c);
    *gr = c;
    *gi = -s;
  } else {
    const float t = (float)(r - rint(r));
    const double c = (double)__builtin_amdgcn_cosf(t);
    const double s = (double)__builtin_amdgcn_sinf(t);
    // One Newton step towards unit modulus: the hardware pair has |g|^2 about
    // 6e-8 below 1 on average, and the binned norm sums are quadratic in g.
    const double k = fma(-0.5, fma(c, c, s * s), 1.5);
    *gr = c * k;
    *gi = -s * k;
  }
}

// Binned sums of one (tile, edge chunk) work item.  The waves of a workgroup
// take consecutive tiles of the same edge chunk; the chunk's edge records are
// staged through LDS in pieces of up to kLdsEdges edges (coalesced copy by the
// whole workgroup, then wave-uniform broadcast reads).  Per lane the partial
// (Z_i, <h_i|h_i>) of the chunk's bins go to ab->part, without the
// (A P_i) / (A0 P0_i) prefactor.
//
// FP64, 20,011 rows of 5000 bins, three detectors: 398 us, of which the vector
// operations (107 an edge and row) take 270 at full rate and LDS 240; 552 us with
// sincos_cycles and every row choosing the edge's weight.  Mixed, 65,536 rows of
// 500 bins: 124 us (145), half of it LDS reads of the records (8 cycles per 16
// bytes, broadcast or not).  Two rows a lane instead of one leave three waves a
// SIMD (584 and 150 us), records as scalar loads wait for them (16,000 rows of
// 5000 bins, mixed: 452 us a call against 396).
constexpr int kLdsEdges = 128;

template <int ND, int PREC>
__global__ void __launch_bounds__(256) k_het(const HetArgs* __restrict__ ab, const int64_t* __restrict__ pre,
                                             const double* __restrict__ rec, int n_bins, int n_ech, TrigConsts T) {
  constexpr int RS = het_rs(ND);
  constexpr int BO = het_bin_off(ND);
  __shared__ double srec[kLdsEdges * RS];
  __shared__ double2 tab[PREC == 0 ? 256 : 1];
  if (PREC == 0) {
    for (int k = threadIdx.x; k < 256; k += blockDim.x) {
      double s, c;
      sincospi((double)k / 128.0, &s, &c);
      tab[k] = make_double2(c, s);
    }
  }
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wpb = blockDim.x >> 6;
  const int64_t total = pre[ab->n_sub];
  const int64_t groups = (total + wpb - 1) / wpb;
  const int64_t ld = ab->ld;
  const double* __restrict__ coef = ab->coef;
  const int per = (n_bins + n_ech - 1) / n_ech;

  for (int64_t q = blockIdx.x; q < groups * n_ech; q += gridDim.x) {
    const int ech = (int)(q % n_ech);
    const int64_t t = (q / n_ech) * wpb + wave;
    int64_t row0 = 0, row_end = 0;
    const bool has = t < total && tile_rows(ab, pre, t, &row0, &row_end);
    const int64_t row = row0 + lane;
    const bool active = has && row < row_end;
    const int64_t rr = active ? row : (has ? row0 : 0);
    const double* cf = coef + rr;
    PhaseCoef c;
    double dt[ND];
    dt[0] = 0.0;
    if (has) {
      c.a0 = cf[C_A0 * ld]; c.a2 = cf[C_A2 * ld]; c.a3 = cf[C_A3 * ld]; c.a4 = cf[C_A4 * ld];
      c.a5 = cf[C_A5 * ld]; c.a6 = cf[C_A6 * ld]; c.a7 = cf[C_A7 * ld]; c.a8 = cf[C_A8 * ld];
      c.a10 = cf[C_A10 * ld]; c.a12 = cf[C_A12 * ld]; c.b5 = cf[C_B5 * ld]; c.b6 = cf[C_B6 * ld];
#pragma unroll
      for (int i = 1; i < ND; ++i) dt[i] = cf[(C_DT1 + i - 1) * ld];
    }

    // bins (b0, b1] of this chunk (bin e lies between edges e - 1 and e) use edges b0 .. b1
    const int b0 = ech * per < n_bins ? ech * per : n_bins;
    const int b1 = b0 + per < n_bins ? b0 + per : n_bins;
    double zr[ND], zi[ND], hh[ND], pr[ND], pi[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      zr[i] = zi[i] = hh[i] = 0.0;
      pr[i] = pi[i] = 0.0;
    }
    const int e_last = b1 > b0 ? b1 : b0 - 1;  // empty chunk: no edges
    for (int e0 = b0; e0 <= e_last; e0 += kLdsEdges) {
      const int ne = e_last - e0 + 1 < kLdsEdges ? e_last - e0 + 1 : kLdsEdges;
      __syncthreads();
      // Edges inside the chunk's bins (b0, b1] weigh C, its first the left-edge
      // part C - R, its last the right-edge part R: set here, not per row (30 of
      // 172 vector operations an edge in FP64)
      for (int j = threadIdx.x; j < ne * RS; j += blockDim.x) {
        const int e = e0 + j / RS, col = j % RS - (BO + 1);
        const double* src = rec + (int64_t)e0 * RS + j;
        double v = *src;
        if ((e == b0 || e == b1) && col >= 0 && col % 6 < 2) v = e == b0 ? v - src[2] : src[2];
        srec[j] = v;
      }
      __syncthreads();
      if (!has) continue;
      for (int el = 0; el < ne; ++el) {
        const double* r = srec + el * RS;
        const double d0 = phase_cycles(c, r[H_X], r[H_X2], r[H_XM5], r[H_LNF]) - r[H_PHI0];
        const double f = r[H_F];
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          double gr, gi;
          const double di = i == 0 ? d0 : fma(f, dt[i], d0) - r[H_PHI0 + i];
          if constexpr (PREC == 0) het_phasor_tab(di, tab, &gr, &gi);
          else het_phasor<PREC>(di, T, &gr, &gi);
          const double* w = r + BO + 1 + 6 * i;
          zr[i] = fma(w[0], gr, fma(-w[1], gi, zr[i]));
          zi[i] = fma(w[0], gi, fma(w[1], gr, zi[i]));
          // |r0|^2 = (1 + Re(g_e conj g_{e-1})) / 2 for unit phasors (no bin
          // ends at the first edge: its predecessor is zero); the constant half
          // is added once per row by the combine kernel
          hh[i] = fma(w[4], fma(gr, pr[i], gi * pi[i]), hh[i]);
          pr[i] = gr;
          pi[i] = gi;
        }
      }
    }
    if (active) {
      double* out = ab->part + (int64_t)ech * 3 * ND * ld + row;
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        out[(3 * i) * ld] = zr[i];
        out[(3 * i + 1) * ld] = zi[i];
        out[(3 * i + 2) * ld] = hh[i];
      }
    }
  }
}

// Combine the edge-chunk partials of each row in chunk order, restore the
// prefactor (A P_i) / (A0 P0_i), sum the detectors and apply the plain or
// phase-marginalised epilogue (or stage |Z_1| and <h|h>_1 for the distance
// marginal).
// Finish one row from its per-detector sums (z_i, unit-phasor <h|h> part):
// restore the prefactor (A P_i) / (A0 P0_i), sum the detectors and apply the
// plain or phase-marginalised epilogue (or stage |Z_1| and <h|h>_1 for the
// distance marginal).
struct HetRow {
  double Zr, Zi, plain, hht;
  bool valid;
};

// A row's binned overlap, its plain real part and <h|h> from the summed edge
// partials (the heterodyne's per-detector ratio to the reference applied).
__device__ inline HetRow het_row(const HetArgs* __restrict__ ab, int64_t row, int nd, const double* zr,
                                 const double* zi, const double* hh, const HetConst& hc) {
  const int64_t ld = ab->ld;
  const double* cf = ab->coef + row;
  double Zr = 0.0, Zi = 0.0, plain = 0.0, hht = 0.0;
  for (int i = 0; i < nd; ++i) {
    const double ar = cf[(C_APRE + i) * ld], ai = cf[(C_APIM + i) * ld];
    const double qr = ar * hc.ap0_inv_re[i] - ai * hc.ap0_inv_im[i];
    const double qi = ar * hc.ap0_inv_im[i] + ai * hc.ap0_inv_re[i];
    const double wr = qr * zr[i] - qi * zi[i];
    const double wi = qr * zi[i] + qi * zr[i];
    plain += wr;
    Zr += wr;
    Zi += wi;
    hht += (qr * qr + qi * qi) * (hc.hh0[i] + hh[i]);
  }
  return HetRow{Zr, Zi, plain, hht, cf[C_VALID * ld] != 0.0};
}

__device__ inline void het_finish_row(const HetArgs* __restrict__ ab, int64_t row, int nd, int marg,
                                      const double* zr, const double* zi, const double* hh, const HetConst& hc) {
  const int64_t ld = ab->ld;
  const HetRow R = het_row(ab, row, nd, zr, zi, hh, hc);
  const double Zr = R.Zr, Zi = R.Zi, plain = R.plain, hht = R.hht;
  const bool valid = R.valid;
  const double zabs = sqrt(Zr * Zr + Zi * Zi);
  if (ab->zcplx) {
    ab->zcplx[row] = valid ? Zr : NAN;
    ab->zcplx[ld + row] = Zi;
    ab->zcplx[2 * ld + row] = hht;
  }
  if (marg == 2) {
    ab->zbuf[row] = valid ? zabs : -1.0;
    ab->zbuf[ld + row] = hht;
  } else {
    double out;
    if (!valid) out = -INFINITY;
    else if (marg == 0) out = -0.5 * hc.dd + plain - 0.5 * hht;
    else out = -0.5 * hc.dd - 0.5 * hht + log_i0(zabs);
    ab->logl[row] = out;
  }
}

// Large batches: a workgroup of four waves per 64-row tile, lane = row; each
// wave sums some of the 3 nd columns over the edge chunks in chunk order, eight
// loads in flight, and wave 0 finishes the rows.  20,011 rows of 53 chunks: 22
// us, 65 with a wave a tile and a load at a time.
__global__ void __launch_bounds__(256) k_het_combine(const HetArgs* __restrict__ ab, const int64_t* __restrict__ pre,
                                                     int nd, int n_ech, int marg, HetConst hc) {
  __shared__ double col[3 * kMaxDet][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t total = pre[ab->n_sub];
  const int64_t ld = ab->ld;
  for (int64_t t = blockIdx.x; t < total; t += gridDim.x) {
    int64_t row0, row_end;
    if (!tile_rows(ab, pre, t, &row0, &row_end)) continue;  // the same for the workgroup
    const int64_t row = row0 + lane < row_end ? row0 + lane : row0;
    const int64_t step = (int64_t)3 * nd * ld;
    for (int c = wave; c < 3 * nd; c += 4) {
      const double* __restrict__ p = ab->part + c * ld + row;
      double s = 0.0;
#pragma unroll 8
      for (int e = 0; e < n_ech; ++e) s += p[e * step];
      col[c][lane] = s;
    }
    __syncthreads();
    if (wave == 0 && row0 + lane < row_end) {
      double zr[kMaxDet], zi[kMaxDet], hh[kMaxDet];
      for (int i = 0; i < nd; ++i) {
        zr[i] = col[3 * i][lane];
        zi[i] = col[3 * i + 1][lane];
        hh[i] = col[3 * i + 2][lane];
      }
      het_finish_row(ab, row, nd, marg, zr, zi, hh, hc);
    }
    __syncthreads();
  }
}

// Small batches (and at most 64 edge chunks): one wave per row, lane e
// holding chunk e's partials, summed by a fixed shuffle tree, so that the
// loads of a row are issued together instead of one chain per thread.
__global__ void __launch_bounds__(256) k_het_combine_w(const HetArgs* __restrict__ ab,
                                                       const int64_t* __restrict__ pre, int nd, int n_ech, int marg,
                                                       HetConst hc) {
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  const int64_t wid = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * wpb;
  const int64_t total = pre[ab->n_sub] * 64;
  const int64_t ld = ab->ld;
  for (int64_t it = wid; it < total; it += nwaves) {
    int64_t row0, row_end;
    if (!tile_rows(ab, pre, it >> 6, &row0, &row_end)) continue;
    const int64_t row = row0 + (it & 63);
    if (row >= row_end) continue;
    double zr[kMaxDet], zi[kMaxDet], hh[kMaxDet];
    for (int i = 0; i < nd; ++i) {
      double a = 0.0, b = 0.0, c = 0.0;
      if (lane < n_ech) {
        const double* p = ab->part + ((int64_t)lane * 3 * nd + 3 * i) * ld + row;
        a = p[0];
        b = p[ld];
        c = p[2 * ld];
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
        c += __shfl_xor(c, o, 64);
      }
      zr[i] = a;
      zi[i] = b;
      hh[i] = c;
    }
    if (lane == 0) het_finish_row(ab, row, nd, marg, zr, zi, hh, hc);
  }
}

// Distance marginal over the work list, small batches and FP64: one wave per row
// (wave_dist_lse), which keeps many waves busy when there are few rows.
template <int PREC>
__global__ void __launch_bounds__(256) k_het_dist_w(const HetArgs* __restrict__ ab, const int64_t* __restrict__ pre,
                                                    const double* __restrict__ dtab, int n_dist, double dd,
                                                    const LogI0Consts* __restrict__ Cp) {
  const LogI0Consts& C = *Cp;
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  const int64_t wid = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * wpb;
  const int64_t total = pre[ab->n_sub] * 64;
  const int64_t ld = ab->ld;
  for (int64_t it = wid; it < total; it += nwaves) {
    int64_t row0, row_end;
    if (!tile_rows(ab, pre, it >> 6, &row0, &row_end)) continue;
    const int64_t row = row0 + (it & 63);
    if (row >= row_end) continue;
    const double z1 = ab->zbuf[row];
    const double h1 = ab->zbuf[ld + row];
    if (z1 < 0.0) {
      if (lane == 0) ab->logl[row] = -INFINITY;
      continue;
    }
    const double v = PREC == 0 ? wave_dist_lse(z1, h1, dtab, n_dist, lane, C)
                               : wave_dist_lse_f32(z1, h1, dtab, n_dist, lane);
    if (lane == 0) ab->logl[row] = -0.5 * dd + v;
  }
}

// Small batches with the distance marginal: k_het_combine_w and k_het_dist_w
// in one launch (one wave per row), the row's |Z| and <h|h> passed on in
// registers; the same arithmetic, so the same log L.
template <int PREC>
__global__ void __launch_bounds__(256) k_het_combine_dist_w(const HetArgs* __restrict__ ab,
                                                            const int64_t* __restrict__ pre, int nd, int n_ech,
                                                            HetConst hc, const double* __restrict__ dtab, int n_dist,
                                                            const LogI0Consts* __restrict__ Cp) {
  const LogI0Consts& C = *Cp;
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  const int64_t wid = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * wpb;
  const int64_t total = pre[ab->n_sub] * 64;
  const int64_t ld = ab->ld;
  for (int64_t it = wid; it < total; it += nwaves) {
    int64_t row0, row_end;
    if (!tile_rows(ab, pre, it >> 6, &row0, &row_end)) continue;
    const int64_t row = row0 + (it & 63);
    if (row >= row_end) continue;
    double zr[kMaxDet], zi[kMaxDet], hh[kMaxDet];
    for (int i = 0; i < nd; ++i) {
      double a = 0.0, b = 0.0, c = 0.0;
      if (lane < n_ech) {
        const double* p = ab->part + ((int64_t)lane * 3 * nd + 3 * i) * ld + row;
        a = p[0];
        b = p[ld];
        c = p[2 * ld];
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
        c += __shfl_xor(c, o, 64);
      }
      zr[i] = a;
      zi[i] = b;
      hh[i] = c;
    }
    const HetRow R = het_row(ab, row, nd, zr, zi, hh, hc);
    const double z1 = R.valid ? sqrt(R.Zr * R.Zr + R.Zi * R.Zi) : -1.0, h1 = R.hht;
    if (lane == 0) {
      if (ab->zcplx) {
        ab->zcplx[row] = R.valid ? R.Zr : NAN;
        ab->zcplx[ld + row] = R.Zi;
        ab->zcplx[2 * ld + row] = R.hht;
      }
      ab->zbuf[row] = z1;
      ab->zbuf[ld + row] = h1;
    }
    if (z1 < 0.0) {
      if (lane == 0) ab->logl[row] = -INFINITY;
      continue;
    }
    const double v = PREC == 0 ? wave_dist_lse(z1, h1, dtab, n_dist, lane, C)
                               : wave_dist_lse_f32(z1, h1, dtab, n_dist, lane);
    if (lane == 0) ab->logl[row] = -0.5 * hc.dd + v;
  }
}

// Distance marginal over the work list, large mixed batches: a workgroup per 64-row
// tile, lane = row, waves splitting the grid (block_dist_lse), so that grid
// records are scalar loads shared by 64 rows.
constexpr int64_t kDistRowsPerLane = 8192;  // batches from this size use the sliced form
constexpr int kHetDistWaves = 8;  // waves per 64-row tile in the sliced form

__global__ void __launch_bounds__(64 * kHetDistWaves) k_het_dist(const HetArgs* __restrict__ ab,
                                                                 const int64_t* __restrict__ pre,
                                                                 const double* __restrict__ dtab, int n_dist,
                                                                 double dd) {
  __shared__ double red[kHetDistWaves * 64];
  const int lane = threadIdx.x & 63;
  const int nw = blockDim.x >> 6;
  const int64_t tiles = pre[ab->n_sub];
  const int64_t ld = ab->ld;
  // one 64-row tile per workgroup iteration (uniform across the block)
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    int64_t row0 = 0, row_end = 0;
    const bool has = tile_rows(ab, pre, t, &row0, &row_end);
    const int64_t row = row0 + lane;
    const bool active = has && row < row_end;
    const int64_t rr = active ? row : (has ? row0 : 0);
    const double z1 = has ? ab->zbuf[rr] : 0.0;
    const double h1 = has ? ab->zbuf[ld + rr] : 0.0;
    const double v = block_dist_lse(z1 < 0.0 ? 0.0 : z1, h1, dtab, n_dist, nw, red);
    if ((threadIdx.x >> 6) == 0 && active) ab->logl[row] = z1 < 0.0 ? -INFINITY : -0.5 * dd + v;
  }
}

// ---------------------------------------------------------------------------
// Host side

static void free_state(gw_het_state* h) {
  if (!h) return;
  if (h->tm_tab) (void)hipFree(h->tm_tab);
  if (h->tm_idx) (void)hipFree(h->tm_idx);
  if (h->rec) (void)hipFree(h->rec);
  if (h->args) (void)hipFree(h->args);
  if (h->tile_pre) (void)hipFree(h->tile_pre);
  if (h->subs_single) (void)hipFree(h->subs_single);
  delete h;
}

void het_free(gw_ctx* ctx) {
  free_state(ctx->het);
  ctx->het = nullptr;
}

static void graphs_clear(gw_graph_cache* g) {
  for (auto& kv : g->exec) (void)hipGraphExecDestroy(kv.second);
  for (auto& kv : g->graph) (void)hipGraphDestroy(kv.second);
  g->exec.clear();
  g->graph.clear();
}

void graphs_free(gw_ctx* ctx) {
  if (!ctx->graphs) return;
  graphs_clear(ctx->graphs);
  if (ctx->graphs->cap_stream) (void)hipStreamDestroy(ctx->graphs->cap_stream);
  delete ctx->graphs;
  ctx->graphs = nullptr;
}

// Edge indices of the bin grid (host, FP64); see heterodyne_setup in gwswig.h.
static std::vector<int64_t> make_edges(const Geom& g, int n_bins, int rule) {
  const int64_t n = g.n_freq;
  std::vector<double> f(n);
  for (int64_t k = 0; k < n; ++k) f[k] = (double)(g.k0 + k) * g.df;
  const double fmin = f[0], fmax = f[n - 1];
  std::vector<double> fe(n_bins + 1);
  if (rule == 0) {
    const double gam[5] = {-5.0 / 3.0, -2.0 / 3.0, 1.0, 5.0 / 3.0, 7.0 / 3.0};
    std::vector<double> phi(n);
    for (int64_t k = 0; k < n; ++k) {
      double s = 0.0;
      for (double gg : gam) {
        const double fs = gg > 0 ? fmax : fmin;
        s += (gg > 0 ? 1.0 : -1.0) * pow(f[k] / fs, gg);
      }
      phi[k] = s;
    }
    int64_t k = 0;
    for (int j = 0; j <= n_bins; ++j) {
      const double y = phi[0] + j * (phi[n - 1] - phi[0]) / n_bins;
      while (k + 1 < n - 1 && phi[k + 1] <= y) ++k;
      if (y <= phi[0]) fe[j] = f[0];
      else if (y >= phi[n - 1]) fe[j] = f[n - 1];
      else fe[j] = f[k] + (y - phi[k]) * (f[k + 1] - f[k]) / (phi[k + 1] - phi[k]);
    }
  } else {
    for (int j = 0; j <= n_bins; ++j) fe[j] = fmin * pow(fmax / fmin, (double)j / n_bins);
  }
  std::vector<int64_t> idx(n_bins + 1);
  for (int j = 0; j <= n_bins; ++j) {
    int64_t v = (int64_t)rint((fe[j] - fmin) / (f[1 < n ? 1 : 0] - f[0] + (n > 1 ? 0.0 : 1.0)));
    idx[j] = std::min<int64_t>(std::max<int64_t>(v, 0), n - 1);
  }
  idx[0] = 0;
  idx[n_bins] = n - 1;
  std::sort(idx.begin(), idx.end());
  idx.erase(std::unique(idx.begin(), idx.end()), idx.end());
  return idx;
}

// Edge chunks per tile: enough (tile, chunk) items to give every SIMD a few
// waves at this batch size, at least 16 bins per chunk, at most 32 chunks.
// Default persistent grid of the evaluation kernel, in waves (measured best
// of 2048 .. 16384 at 65,536 rows and 500 bins).
constexpr int64_t kHetWaves = 16384;

static int het_ech(const gw_ctx* ctx, int64_t n_rows) {
  const int64_t nb = ctx->het->n_bins;
  if (ctx->het->ech > 0) return (int)std::min<int64_t>(ctx->het->ech, nb);
  // about one (tile, edge chunk) item per wave of the default grid, at most
  // 64 chunks (one lane each in the combine) of at least 8 edges: a
  // sampler's 250-row batch of 500 bins takes 31.2 us a call at 62 chunks
  // against 36.0 at 31
  // Large batches take at least 48 bins a chunk: its start and its partials
  // (three per detector and row) weigh more than the waves it adds (mixed, 500
  // bins: 12,000 rows 109 us at 62 chunks and 84 at 10, 30,000 rows 141 at 35
  // and 133 at 10); but with few bins as many as make 1024 items, one a SIMD, of
  // at least 12 bins (FP64, 9000 rows: 50 bins 41 us in one chunk, 28 in four;
  // 100 bins 42 in two, 30 in eight).
  const int64_t tiles = (n_rows + 63) / 64;
  int64_t e = (kHetWaves + tiles - 1) / tiles;
  int64_t emax = std::min<int64_t>(64, nb / 8);
  if (n_rows >= kDistRowsPerLane) emax = std::min<int64_t>(64, std::max(nb / 48, std::min(nb / 12, 1024 / tiles)));
  emax = std::max<int64_t>(1, emax);
  e = std::max<int64_t>(1, std::min(e, emax));
  return (int)e;
}

template <int ND>
static gw_status launch_het_nd(gw_ctx* ctx, int marg, int prec, int n_ech, hipStream_t st) {
  gw_het_state* h = ctx->het;
  const TrigConsts T = make_trig_consts();
  const int tpb = 64 * h->wpb;
  int grid = h->grid;
  // 64 waves per CU (several rounds of the resident 20); small batches have
  // few items, and an idle grid still costs dispatch time
  if (grid <= 0) grid = (h->n_rows_last < kDistRowsPerLane ? 1024 : kHetWaves) / h->wpb;
  const int slot = prof_begin(ctx, st, 1);
  if (prec == GW_PREC_FP64)
    hipLaunchKernelGGL((k_het<ND, 0>), dim3(grid), dim3(tpb), 0, st, h->args, h->tile_pre, h->rec, h->n_bins, n_ech,
                       T);
  else
    hipLaunchKernelGGL((k_het<ND, 1>), dim3(grid), dim3(tpb), 0, st, h->args, h->tile_pre, h->rec, h->n_bins, n_ech,
                       T);
  prof_end(ctx, slot, st);
  (void)marg;
  return check_hip(hipGetLastError(), "heterodyne kernel launch");
}

// Queue the work-list sequence: tile scan, prologue, binned sums, combine
// (+ distance marginal).  Reads the device argument block only.
static gw_status enqueue_het(gw_ctx* ctx, int marg, int prec, int n_ech, hipStream_t st) {
  gw_het_state* h = ctx->het;
  const bool small = h->n_rows_last < kDistRowsPerLane;
  hipLaunchKernelGGL(k_het_prologue, dim3(small ? 128 : 256 * 4), dim3(128), 0, st, h->args, h->tile_pre, marg,
                     ctx->geom);
  gw_status s = check_hip(hipGetLastError(), "heterodyne prologue launch");
  if (s != GW_OK) return s;
  switch (ctx->n_det) {
    case 1: s = launch_het_nd<1>(ctx, marg, prec, n_ech, st); break;
    case 2: s = launch_het_nd<2>(ctx, marg, prec, n_ech, st); break;
    case 3: s = launch_het_nd<3>(ctx, marg, prec, n_ech, st); break;
    case 4: s = launch_het_nd<4>(ctx, marg, prec, n_ech, st); break;
    default: s = set_error(GW_ENOTSUP, "n_det not supported");
  }
  if (s != GW_OK) return s;
  HetConst hc;
  for (int i = 0; i < kMaxDet; ++i) {
    hc.ap0_inv_re[i] = h->ap0_inv_re[i];
    hc.ap0_inv_im[i] = h->ap0_inv_im[i];
    hc.hh0[i] = h->hh0[i];
  }
  hc.dd = ctx->dd;
  if (marg == 2 && h->n_rows_last < kDistRowsPerLane && n_ech <= 64) {
    if (prec == GW_PREC_MIXED)
      hipLaunchKernelGGL(k_het_combine_dist_w<1>, dim3(256 * 8), dim3(256), 0, st, h->args, h->tile_pre, ctx->n_det,
                         n_ech, hc, ctx->dist_tab, ctx->n_dist, ctx->i0c);
    else
      hipLaunchKernelGGL(k_het_combine_dist_w<0>, dim3(256 * 8), dim3(256), 0, st, h->args, h->tile_pre, ctx->n_det,
                         n_ech, hc, ctx->dist_tab, ctx->n_dist, ctx->i0c);
    return check_hip(hipGetLastError(), "heterodyne combine and distance marginal launch");
  }
  if (h->n_rows_last < kDistRowsPerLane && n_ech <= 64)
    hipLaunchKernelGGL(k_het_combine_w, dim3(256 * 8), dim3(256), 0, st, h->args, h->tile_pre, ctx->n_det, n_ech,
                       marg, hc);
  else
    hipLaunchKernelGGL(k_het_combine, dim3(256 * 8), dim3(256), 0, st, h->args, h->tile_pre, ctx->n_det, n_ech,
                       marg, hc);
  s = check_hip(hipGetLastError(), "heterodyne combine launch");
  if (s != GW_OK || marg != 2) return s;
  // large mixed batches: lane = row (grid records are scalar loads shared by
  // 64 rows).  Small ones and FP64: wave = row; its lanes are neighbouring
  // distances, which take the same form of a term (skipped, FP32, series or
  // asymptotic), while rows differ: 20,011 rows in FP64 take 85 us against 230
  if (h->n_rows_last >= kDistRowsPerLane && prec == GW_PREC_MIXED)
    hipLaunchKernelGGL(k_het_dist, dim3(256 * 8), dim3(64 * kHetDistWaves), 0, st, h->args, h->tile_pre,
                       ctx->dist_tab, ctx->n_dist, ctx->dd);
  else if (prec == GW_PREC_MIXED)
    hipLaunchKernelGGL(k_het_dist_w<1>, dim3(256 * 8), dim3(256), 0, st, h->args, h->tile_pre, ctx->dist_tab,
                       ctx->n_dist, ctx->dd, ctx->i0c);
  else
    hipLaunchKernelGGL(k_het_dist_w<0>, dim3(256 * 8), dim3(256), 0, st, h->args, h->tile_pre, ctx->dist_tab,
                       ctx->n_dist, ctx->dd, ctx->i0c);
  return check_hip(hipGetLastError(), "heterodyne distance marginal launch");
}

// Workspace for n_rows rows and the argument block; returns the edge-chunk count.
static gw_status het_prepare(gw_ctx* ctx, const double* theta, const int64_t* subs, int32_t n_sub, int64_t n_rows,
                             double* logl, bool single, int* n_ech, hipStream_t st, double* zcplx = nullptr) {
  gw_het_state* h = ctx->het;
  h->n_rows_last = n_rows;
  *n_ech = het_ech(ctx, n_rows);
  gw_status s = ensure_buffer(&ctx->coef, &ctx->coef_cap, (int64_t)C_NCOEF * n_rows, "coefficient workspace");
  if (s == GW_OK) s = ensure_buffer(&ctx->zbuf, &ctx->zbuf_cap, 2 * n_rows, "marginal workspace");
  if (s == GW_OK)
    s = ensure_buffer(&ctx->partial, &ctx->partial_cap, (int64_t)(*n_ech) * 3 * ctx->n_det * n_rows, "partials");
  if (s != GW_OK) return s;
  if (h->args_pinned) {
    if (single && !zcplx && theta == h->pin_theta && logl == h->pin_logl && n_rows == h->pin_rows) return GW_OK;
    h->args_pinned = false;  // the block is rewritten below
  }
  hipLaunchKernelGGL(k_set_args, dim3(1), dim3(256), 0, st, h->args, theta,
                     single ? (const int64_t*)h->subs_single : subs, logl, ctx->coef, ctx->zbuf, ctx->partial, n_rows,
                     single ? 1 : n_sub, single ? h->subs_single : (int64_t*)nullptr, single ? n_rows : (int64_t)0,
                     h->tile_pre, zcplx);
  return check_hip(hipGetLastError(), "argument kernel launch");
}

gw_status het_pin_args(gw_ctx* ctx, const double* theta, int64_t n, double* logl, hipStream_t st) {
  gw_het_state* h = ctx->het;
  if (!h) return set_error(GW_ESTATE, "heterodyne_setup has not been called");
  h->args_pinned = false;
  int n_ech = 1;
  gw_status s = het_prepare(ctx, theta, nullptr, 1, n, logl, true, &n_ech, st);
  if (s != GW_OK) return s;
  h->pin_theta = theta;
  h->pin_logl = logl;
  h->pin_rows = n;
  h->args_pinned = true;
  return GW_OK;
}

void het_unpin_args(gw_ctx* ctx) {
  if (ctx->het) ctx->het->args_pinned = false;
}

gw_status het_reserve(gw_ctx* ctx, int64_t n) {
  if (!ctx->het) return set_error(GW_ESTATE, "heterodyne_setup has not been called");
  const int n_ech = het_ech(ctx, n);
  gw_status s = ensure_buffer(&ctx->coef, &ctx->coef_cap, (int64_t)C_NCOEF * n, "coefficient workspace");
  if (s == GW_OK) s = ensure_buffer(&ctx->zbuf, &ctx->zbuf_cap, 2 * n, "marginal workspace");
  if (s == GW_OK) s = ensure_buffer(&ctx->partial, &ctx->partial_cap, (int64_t)n_ech * 3 * ctx->n_det * n, "partials");
  return s;
}

void het_shape_key(const gw_ctx* ctx, int32_t* wpb, int32_t* grid, int32_t* ech) {
  *wpb = ctx->het ? ctx->het->wpb : 0;
  *grid = ctx->het ? ctx->het->grid : 0;
  *ech = ctx->het ? ctx->het->ech : 0;
}

void het_tm_key(const gw_ctx* ctx, const void** tab, const void** idx, int32_t* nch) {
  const gw_het_state* h = ctx->het;
  *tab = h ? h->tm_tab : nullptr;
  *idx = h ? h->tm_idx : nullptr;
  *nch = h ? h->tm_nch : 0;
}

// ---------------------------------------------------------------------------
// Time marginal on the binned likelihood (the appendix's direct sum on the
// heterodyned bins).  A shift t multiplies every edge phasor by
// exp(-2 pi i f_e t), so with per-row edge weights
//   W_e = sum_i q_i K_ie g_ie          (K the summed-by-parts overlap weights),
//   V_e = sum_i |q_i|^2 (B0_e / 2) g_ie conj(g_i,e-1)   (bin e's norm term),
// q_i = (A P_i) / (A0 P0_i), the binned overlap and norm at t_j are
//   Z(t_j)  = sum_e W_e exp(-2 pi i f_e t_j),
//   hh(t_j) = sum_i |q_i|^2 hh0_i + Re sum_e V_e exp(-2 pi i (f_e - f_e-1) t_j).
// The edges lie on the fine grid, so Z goes through the frequency grid of the
// full band's time marginal with W_e in place of the per-bin weights
// (gw_tgrid.hip); the widths f_e - f_e-1 = dk_e df span a short range, and
// exp(-2 pi i dk_e u) about the widths' centre c, dk_e = c + hw sigma_e, is a
// series in (2 pi hw u) sigma_e whose moments S_m = sum_e sigma_e^m V_e the
// grid kernel sums (tm_mh terms, the first dropped one below 1e-13 of
// sum_e |V_e| at the window's edge).

// Sums over the edges of one (64-row tile, chunk): lane = row, the chunk's
// edges e0[c] .. e0[c + 1] in order (edge records and tables wave-uniform).
// GRID: W spread onto the grid, the window of kTgW points sliding over the
// chunk's cells (a point that no later edge reaches is stored), into part
// [rows][pitch]; chunk 0 also writes the constant norm part hhc [rows].  Both
// forms: S_m, m0 <= m < m0 + MH (m < mh), over the chunk's edges into hpart
// [chunk][rows][mh].  The GRID form takes the first moments along, which
// spares their phases and phasors (mixed, 5000 bins: 32 us for both at 128 rows,
// 36 + 21 in two passes).
template <int ND, int PREC, bool GRID, int MH>
__global__ void __launch_bounds__(64) k_het_tmom(const double* __restrict__ coef, int64_t ld, int64_t n,
                                                 const double* __restrict__ rec, int n_bins,
                                                 const double* __restrict__ tab, int mh,
                                                 const int32_t* __restrict__ cell, const int32_t* __restrict__ plan,
                                                 int nch, int m0, HetConst hc, TrigConsts T, int64_t pitch,
                                                 double2* __restrict__ part, double2* __restrict__ hpart,
                                                 double* __restrict__ hhc) {
  constexpr int K = kTgW;
  constexpr int RS = het_rs(ND);
  constexpr int BO = het_bin_off(ND);
  const int64_t p = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int64_t pc = p < n ? p : n - 1;
  const int ch = blockIdx.y;
  const double* cf = coef + pc;
  PhaseCoef c;
  c.a0 = cf[C_A0 * ld]; c.a2 = cf[C_A2 * ld]; c.a3 = cf[C_A3 * ld]; c.a4 = cf[C_A4 * ld];
  c.a5 = cf[C_A5 * ld]; c.a6 = cf[C_A6 * ld]; c.a7 = cf[C_A7 * ld]; c.a8 = cf[C_A8 * ld];
  c.a10 = cf[C_A10 * ld]; c.a12 = cf[C_A12 * ld]; c.b5 = cf[C_B5 * ld]; c.b6 = cf[C_B6 * ld];
  double dt[ND], qr[ND], qi[ND], q2[ND], pr[ND], pim[ND];
  double hconst = 0.0;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    dt[i] = i == 0 ? 0.0 : cf[(C_DT1 + i - 1) * ld];
    const double ar = cf[(C_APRE + i) * ld], ai = cf[(C_APIM + i) * ld];
    qr[i] = ar * hc.ap0_inv_re[i] - ai * hc.ap0_inv_im[i];
    qi[i] = ar * hc.ap0_inv_im[i] + ai * hc.ap0_inv_re[i];
    q2[i] = qr[i] * qr[i] + qi[i] * qi[i];
    hconst = fma(q2[i], hc.hh0[i], hconst);
    pr[i] = pim[i] = 0.0;
  }
  if (GRID && ch == 0 && p < n) hhc[p] = hconst;
  const int32_t* __restrict__ e0 = plan;
  const int e_lo = e0[ch], e_hi = e0[ch + 1];
  const int tw_ = K + mh;  // table row length
  if (e_lo > 0) {  // the norm term needs the previous edge's phasors
    const double* r = rec + (int64_t)(e_lo - 1) * RS;
    const double d0 = phase_cycles(c, r[H_X], r[H_X2], r[H_XM5], r[H_LNF]) - r[H_PHI0];
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const double di = i == 0 ? d0 : fma(r[H_F], dt[i], d0) - r[H_PHI0 + i];
      het_phasor<PREC>(di, T, &pr[i], &pim[i]);
    }
  }
  double ar_[K], ai_[K], hr[MH], hi[MH];
#pragma unroll
  for (int m = 0; m < K; ++m) ar_[m] = ai_[m] = 0.0;
#pragma unroll
  for (int m = 0; m < MH; ++m) hr[m] = hi[m] = 0.0;
  double2* out = part + p * pitch;
  int cur = 0;  // the window's first grid point
  auto slide = [&](int to) {
    for (; cur < to; ++cur, ++out) {
      if (p < n) *out = make_double2(ar_[0], ai_[0]);
#pragma unroll
      for (int m = 0; m + 1 < K; ++m) {
        ar_[m] = ar_[m + 1];
        ai_[m] = ai_[m + 1];
      }
      ar_[K - 1] = ai_[K - 1] = 0.0;
    }
  };
  // one edge: W_e onto the grid, V_e into the moments
  auto edge = [&](int e) {
    const double* r = rec + (int64_t)e * RS;
    const double d0 = phase_cycles(c, r[H_X], r[H_X2], r[H_XM5], r[H_LNF]) - r[H_PHI0];
    const double f = r[H_F];
    double wr = 0.0, wi = 0.0, vr = 0.0, vi = 0.0;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const double di = i == 0 ? d0 : fma(f, dt[i], d0) - r[H_PHI0 + i];
      double gr, gi;
      het_phasor<PREC>(di, T, &gr, &gi);
      const double* w = r + BO + 1 + 6 * i;
      if constexpr (GRID) {
        // summed-by-parts weights; the first and last edges take one side
        const double kr = e == 0 ? w[0] - w[2] : (e == n_bins ? w[2] : w[0]);
        const double ki = e == 0 ? w[1] - w[3] : (e == n_bins ? w[3] : w[1]);
        const double kgr = kr * gr - ki * gi, kgi = kr * gi + ki * gr;  // q K g
        wr = fma(qr[i], kgr, fma(-qi[i], kgi, wr));
        wi = fma(qr[i], kgi, fma(qi[i], kgr, wi));
      }
      const double sq = e > 0 ? q2[i] * w[4] : 0.0;  // |q|^2 (B0 / 2) g_e conj(g_e-1)
      vr = fma(sq, fma(gr, pr[i], gi * pim[i]), vr);
      vi = fma(sq, fma(gi, pr[i], -gr * pim[i]), vi);
      pr[i] = gr;
      pim[i] = gi;
    }
    const double* tp = tab + (int64_t)e * tw_;
    if constexpr (GRID) {
      slide(cell[e]);
#pragma unroll
      for (int m = 0; m < K; ++m) {
        ar_[m] = fma(tp[m], wr, ar_[m]);
        ai_[m] = fma(tp[m], wi, ai_[m]);
      }
    }
    tp += K + m0;
#pragma unroll
    for (int m = 0; m < MH; ++m) {
      const double t = m0 + m < mh ? tp[m] : 0.0;
      hr[m] = fma(t, vr, hr[m]);
      hi[m] = fma(t, vi, hi[m]);
    }
  };
  const int32_t* __restrict__ blo = e0 + nch + 1;
  const int32_t* __restrict__ bhi = blo + nch;
  if (GRID) {
    cur = blo[ch];
    out += (bhi + nch)[ch];
  }
  for (int e = e_lo; e < e_hi; ++e) edge(e);
  if (GRID) slide(bhi[ch] - 1);
  if (p < n) {
    if (GRID) {
#pragma unroll
      for (int m = 0; m < K; ++m) out[m] = make_double2(ar_[m], ai_[m]);
    }
    double2* ho = hpart + ((int64_t)ch * n + p) * mh + m0;
#pragma unroll
    for (int m = 0; m < MH; ++m)
      if (m0 + m < mh) ho[m] = make_double2(hr[m], hi[m]);
  }
}

template <int ND>
static void launch_het_tmom_nd(gw_ctx* ctx, const double* coef, int64_t ld, int64_t n, int prec, const HetConst& hc,
                               double2* part, double2* hpart, double* hhc, hipStream_t st) {
  const gw_het_state* h = ctx->het;
  const dim3 grid((unsigned)((n + 63) / 64), (unsigned)h->tm_nch);
  auto launch = [&](auto kernel, int m0) {
    hipLaunchKernelGGL(kernel, grid, dim3(64), 0, st, coef, ld, n, (const double*)h->rec, h->n_bins,
                       (const double*)h->tm_tab, h->tm_mh, h->tm_cell, h->tm_cell + h->n_edges, h->tm_nch, m0, hc,
                       make_trig_consts(), (int64_t)h->tm_npts, part, hpart, hhc);
  };
  const bool fp64 = prec == GW_PREC_FP64;
  if (h->tm_mh <= 8)
    fp64 ? launch(k_het_tmom<ND, 0, true, 8>, 0) : launch(k_het_tmom<ND, 1, true, 8>, 0);
  else
    fp64 ? launch(k_het_tmom<ND, 0, true, 14>, 0) : launch(k_het_tmom<ND, 1, true, 14>, 0);
  for (int m0 = 14; m0 < h->tm_mh; m0 += 14)
    fp64 ? launch(k_het_tmom<ND, 0, false, 14>, m0) : launch(k_het_tmom<ND, 1, false, 14>, m0);
}

// Chunks of the moment kernel: edge ranges of about equal cost (an edge or
// a cell's store count one unit each; gw_hetplan.h), the count
// chosen for about 4096 (tile, chunk) waves (at most 256 chunks, each of at
// least 8 units), or fixed by gw_set_het_tm_split.
static int het_tm_chunks(const gw_ctx* ctx, int64_t n, int n_cell) {
  if (ctx->tm_nsk > 0) return ctx->tm_nsk;
  const int64_t tiles = (n + 63) / 64;
  int64_t want = (4096 + tiles - 1) / tiles;
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>(256, (ctx->het->n_edges + n_cell) / 8));
  return (int)std::max<int64_t>(1, std::min(want, most));
}

// Row-independent tables of the time marginal for the grid and nch edge chunks.
static gw_status het_tm_tables(gw_ctx* ctx, const TimeGridShape& g, int nch) {
  gw_het_state* h = ctx->het;
  if (h->tm_tab && h->tm_blk == g.blk && h->tm_nblk == g.n_blk && h->tm_nch_req == nch && h->tm_L == g.L &&
      h->tm_jmax == g.jmax)
    return GW_OK;
  const double umax = (double)g.jmax / ((double)g.N * (double)g.R);  // the window's largest |u|, fine-grid cycles
  const int n_cell = 2 * g.n_blk;
  const int ne = h->n_edges;
  std::vector<int64_t> k(ne);
  for (int e = 0; e < ne; ++e) k[e] = (int64_t)llround(h->f_edges[e] / ctx->geom.df) - ctx->geom.k0;
  int64_t dmin = INT64_MAX, dmax = 0;
  for (int e = 1; e < ne; ++e) {
    dmin = std::min(dmin, k[e] - k[e - 1]);
    dmax = std::max(dmax, k[e] - k[e - 1]);
  }
  if (ne < 2) dmin = dmax = 0;
  const double cw = 0.5 * (double)(dmin + dmax), hw = 0.5 * (double)(dmax - dmin);
  // norm series length: (x^M / M!) e^x below 1e-13, x = 2 pi hw umax
  const double x = 2.0 * kPi * hw * umax;
  int mh = 1;
  double term = x;
  while (term * exp(x) > 1e-13 && mh < kTgHMax) {
    ++mh;
    term *= x / (double)mh;
  }
  if (term * exp(x) > 1e-13)
    return set_error(GW_ENOTSUP, "heterodyned time marginal: bin widths up to %lld fine bins over a +-%.3g s window "
                                 "need more than %d norm terms", (long long)dmax, ctx->tm_window, kTgHMax);
  const int tw_ = kTgW + mh;
  std::vector<double> tab((size_t)ne * tw_, 0.0);
  std::vector<int32_t> cs(n_cell + 1, 0), cell(ne);
  const TgWindow win(g.beta);
  for (int e = 0; e < ne; ++e) {
    const double x = (double)k[e] / g.cell;
    if (k[e] < 0 || x >= n_cell) return set_error(GW_EINVAL, "heterodyned time marginal: edge outside the band");
    cell[e] = (int32_t)x;
    cs[cell[e] + 1] += 1;
    win.weights(x - cell[e], tab.data() + (size_t)e * tw_);
    const double sg = e > 0 && hw > 0.0 ? ((double)(k[e] - k[e - 1]) - cw) / hw : 0.0;
    double tp = 1.0;
    for (int m = 0; m < mh; ++m) {
      tab[(size_t)e * tw_ + kTgW + m] = tp;
      tp *= sg;
    }
  }
  for (int b = 0; b < n_cell; ++b) cs[b + 1] += cs[b];
  const HetTmPlan plan = het_tm_plan(cs, n_cell, ne, nch);
  std::vector<int32_t> len(plan.nch());
  for (int c = 0; c < plan.nch(); ++c) len[c] = plan.bhi[c] - plan.blo[c] + kTgW - 1;
  const TgCoverPlan cov = tgrid_cover(plan.blo, len, g.n_g);
  std::vector<int32_t> idx(cov.pts), first(plan.nch());
  for (int c = 0; c < plan.nch(); ++c) first[c] = cov.shift[c] + plan.blo[c];
  const std::vector<int32_t>* parts[] = {&cell, &plan.e0, &plan.blo, &plan.bhi, &first, &cov.shift};
  for (const std::vector<int32_t>* v : parts) idx.insert(idx.end(), v->begin(), v->end());
  if (h->tm_tab) (void)hipFree(h->tm_tab);
  if (h->tm_idx) (void)hipFree(h->tm_idx);
  h->tm_tab = nullptr;
  h->tm_idx = nullptr;
  gw_status s = check_hip(hipMalloc((void**)&h->tm_tab, tab.size() * sizeof(double)), "time-marginal tables");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&h->tm_idx, idx.size() * sizeof(int32_t)), "time-marginal index");
  if (s == GW_OK) s = fault_tables("time-marginal tables");
  if (s == GW_OK)
    s = check_hip(hipMemcpy(h->tm_tab, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice), "tables");
  if (s == GW_OK)
    s = check_hip(hipMemcpy(h->tm_idx, idx.data(), idx.size() * sizeof(int32_t), hipMemcpyHostToDevice), "index");
  if (s != GW_OK) {  // no tables: a half of them would pass for the last grid's
    if (h->tm_tab) (void)hipFree(h->tm_tab);
    if (h->tm_idx) (void)hipFree(h->tm_idx);
    h->tm_tab = nullptr;
    h->tm_idx = nullptr;
    return s;
  }
  h->tm_cov = TgCover{(const int4*)h->tm_idx, h->tm_idx + idx.size() - cov.shift.size(), cov.n_many};
  h->tm_cell = h->tm_idx + cov.pts.size();
  h->tm_blk = g.blk;
  h->tm_nblk = g.n_blk;
  h->tm_L = g.L;
  h->tm_jmax = g.jmax;
  h->tm_mh = mh;
  h->tm_nch = plan.nch();
  h->tm_nch_req = nch;
  h->tm_npts = cov.n_pts;
  h->tm_hw = hw;
  h->tm_c2 = dmin + dmax;
  return GW_OK;
}

gw_status loglike_het_tmarg(gw_ctx* ctx, const double* theta, int64_t n, int prec, double* logl, hipStream_t st) {
  return loglike_het_tmarg_staged(ctx, theta, n, prec, logl, nullptr, st);
}

gw_status loglike_het_tmarg_staged(gw_ctx* ctx, const double* theta, int64_t n, int prec, double* logl, double* zout,
                                   hipStream_t st) {
  gw_het_state* h = ctx->het;
  if (!h) return set_error(GW_ESTATE, "loglike_batch: heterodyne_setup has not been called");
  TimeGridShape g;
  gw_status s = time_grid_shape(ctx, &g);
  if (s == GW_OK) s = tgrid_tables(ctx, g.L, g.jmax);
  if (s != GW_OK) return s;
  // rows per chunk for at most one wave of every chunk's window over each cell,
  // edge chunks sized for the rows of one launch
  const int64_t chunk = tgrid_chunk_rows(n, (int64_t)(kTgW + 1) * g.n_blk);
  s = het_tm_tables(ctx, g, het_tm_chunks(ctx, chunk, 2 * g.n_blk));
  if (s != GW_OK) return s;
  const int mh = h->tm_mh;
  // workspace: coefficients for all rows; per row chunk the grid sums
  // [rows][points], the norm moments [n_ch][rows][mh] and hhc [rows]
  s = ensure_buffer(&ctx->coef, &ctx->coef_cap, (int64_t)C_NCOEF * n, "coefficient workspace");
  if (s == GW_OK)
    s = ensure_buffer(&ctx->tm_mom, &ctx->tm_mom_cap,
                      chunk * h->tm_npts * 2 + (int64_t)h->tm_nch * chunk * mh * 2 + chunk,
                      "time-marginal workspace");
  if (s != GW_OK || !theta) return s;  // theta NULL: reserve only
  double2* part = (double2*)ctx->tm_mom;
  double2* hpart = part + chunk * h->tm_npts;
  double* hhc = (double*)(hpart + (int64_t)h->tm_nch * chunk * mh);
  s = launch_prologue(ctx, theta, n, GW_MARG_PHASE_TIME, ctx->coef, n, st, false);
  if (s != GW_OK) return s;
  HetConst hc;
  for (int i = 0; i < kMaxDet; ++i) {
    hc.ap0_inv_re[i] = h->ap0_inv_re[i];
    hc.ap0_inv_im[i] = h->ap0_inv_im[i];
    hc.hh0[i] = h->hh0[i];
  }
  hc.dd = ctx->dd;
  const int nt = 2 * g.jmax + 1;
  for (int64_t r0 = 0; r0 < n && s == GW_OK; r0 += chunk) {
    const int64_t cn = n - r0 < chunk ? n - r0 : chunk;
    const int prof = prof_begin(ctx, st, 1);
    switch (ctx->n_det) {
      case 1: launch_het_tmom_nd<1>(ctx, ctx->coef + r0, n, cn, prec, hc, part, hpart, hhc, st); break;
      case 2: launch_het_tmom_nd<2>(ctx, ctx->coef + r0, n, cn, prec, hc, part, hpart, hhc, st); break;
      case 3: launch_het_tmom_nd<3>(ctx, ctx->coef + r0, n, cn, prec, hc, part, hpart, hhc, st); break;
      case 4: launch_het_tmom_nd<4>(ctx, ctx->coef + r0, n, cn, prec, hc, part, hpart, hhc, st); break;
      default: return set_error(GW_ENOTSUP, "n_det not supported");
    }
    s = check_hip(hipGetLastError(), "time-marginal moment launch");
    if (s != GW_OK) return s;
    prof_end(ctx, prof, st);
    TGridArgs a{};
    a.part = (const double*)part;
    a.pitch = h->tm_npts;
    a.cov[0] = a.cov[1] = h->tm_cov;  // one cover for all rows
    a.n = cn;
    a.n_g = g.n_g;
    a.L = g.L;
    a.jmax = g.jmax;
    a.coef = ctx->coef + r0;
    a.ld = n;
    a.logl = logl + r0;
    a.het = 1;
    a.hhc = hhc;
    a.hpart = (const double*)hpart;
    a.n_hch = h->tm_nch;
    a.mh = mh;
    a.hw_step = 2.0 * kPi * h->tm_hw / ((double)g.N * (double)g.R);
    a.c2 = h->tm_c2;
    a.cden = 2 * g.N * (int64_t)g.R;
    a.zout = zout ? zout + r0 * nt * 3 : nullptr;
    a.f0_num = g.f0_num;
    a.f0_den = g.f0_den;
    const int gslot = prof_begin(ctx, st, 2);
    s = launch_tgrid(ctx, a, st);
    prof_end(ctx, gslot, st);
  }
  return s;
}

gw_status loglike_het(gw_ctx* ctx, const double* theta, int64_t n, int marg, int prec, double* logl, hipStream_t st) {
  if (!ctx->het) return set_error(GW_ESTATE, "loglike_batch: heterodyne_setup has not been called");
  if (marg == GW_MARG_PHASE_TIME) return loglike_het_tmarg(ctx, theta, n, prec, logl, st);
  return loglike_het_staged(ctx, theta, n, marg, prec, logl, nullptr, st);
}

gw_status loglike_het_staged(gw_ctx* ctx, const double* theta, int64_t n, int marg, int prec, double* logl,
                             double* zc3, hipStream_t st) {
  if (!ctx->het) return set_error(GW_ESTATE, "heterodyne_setup has not been called");
  int n_ech = 1;
  gw_status s = het_prepare(ctx, theta, nullptr, 1, n, logl, true, &n_ech, st, zc3);
  if (s != GW_OK) return s;
  return enqueue_het(ctx, marg, prec, n_ech, st);
}

}  // namespace gw

using namespace gw;

extern "C" {

gw_status heterodyne_setup(gw_ctx* ctx, const double* theta0, int32_t n_bins, int32_t bin_rule, double* edges_out) {
  if (!ctx) return set_error(GW_EINVAL, "heterodyne_setup: ctx is NULL");
  if (!theta0) return set_error(GW_EINVAL, "heterodyne_setup: theta0 is NULL");
  if (bin_rule != 0 && bin_rule != 1) return set_error(GW_EINVAL, "heterodyne_setup: bin_rule must be 0 or 1");
  if (n_bins < 1 || (int64_t)n_bins > ctx->geom.n_freq - 1)
    return set_error(GW_EINVAL, "heterodyne_setup: n_bins must be in 1 .. n_freq - 1");
  for (int j = 0; j < 13; ++j)
    if (!isfinite(theta0[j])) return set_error(GW_EINVAL, "heterodyne_setup: theta0 must be finite");
  if (!(theta0[0] > 0.0) || !(theta0[1] > 0.0) || theta0[1] > 1.0 || fabs(theta0[2]) >= 1.0 ||
      fabs(theta0[3]) >= 1.0 || !(theta0[6] > 0.0))
    return set_error(GW_EINVAL, "heterodyne_setup: theta0 is unphysical");
  gw_status s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s != GW_OK) return s;
  het_free(ctx);
  if (ctx->graphs) graphs_clear(ctx->graphs);

  const int nd = ctx->n_det;
  const int64_t nf = ctx->geom.n_freq;
  std::vector<int64_t> edges = make_edges(ctx->geom, n_bins, bin_rule);
  const int ne = (int)edges.size();
  gw_het_state* h = new (std::nothrow) gw_het_state();
  if (!h) return set_error(GW_ENOMEM, "heterodyne_setup: host allocation");
  h->n_edges = ne;
  h->n_bins = ne - 1;
  h->rs = het_rs(nd);
  h->theta0.assign(theta0, theta0 + 13);
  h->max_sub = kMaxSub;
  h->f_edges.resize(ne);
  for (int e = 0; e < ne; ++e) h->f_edges[e] = (double)(ctx->geom.k0 + edges[e]) * ctx->geom.df;

  // hh weights 4 df f^(-7/3) / S for the set-up sums
  std::vector<double> hw((size_t)nd * nf);
  for (int i = 0; i < nd; ++i)
    for (int64_t k = 0; k < nf; ++k) {
      const double f = (double)(ctx->geom.k0 + k) * ctx->geom.df;
      hw[(size_t)i * nf + k] = 4.0 * ctx->geom.df * pow(f, -7.0 / 3.0) / ctx->h_psd[(size_t)i * nf + k];
    }
  double *d_hw = nullptr, *d_th = nullptr, *d_coef0 = nullptr;
  int64_t* d_edges = nullptr;
  auto cleanup = [&]() {
    if (d_hw) (void)hipFree(d_hw);
    if (d_th) (void)hipFree(d_th);
    if (d_coef0) (void)hipFree(d_coef0);
    if (d_edges) (void)hipFree(d_edges);
  };
  s = check_hip(hipMalloc((void**)&d_hw, hw.size() * sizeof(double)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&d_th, 13 * sizeof(double)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&d_coef0, C_NCOEF * sizeof(double)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&d_edges, ne * sizeof(int64_t)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&h->rec, (size_t)ne * h->rs * sizeof(double)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&h->args, sizeof(HetArgs)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&h->tile_pre, (kMaxSub + 1) * sizeof(int64_t)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&h->subs_single, 2 * sizeof(int64_t)), "het alloc");
  if (s == GW_OK) s = check_hip(hipMemcpy(d_hw, hw.data(), hw.size() * sizeof(double), hipMemcpyHostToDevice), "copy");
  if (s == GW_OK) s = check_hip(hipMemcpy(d_th, theta0, 13 * sizeof(double), hipMemcpyHostToDevice), "copy");
  if (s == GW_OK)
    s = check_hip(hipMemcpy(d_edges, edges.data(), ne * sizeof(int64_t), hipMemcpyHostToDevice), "copy");
  if (s == GW_OK) s = check_hip(hipMemset(h->rec, 0, (size_t)ne * h->rs * sizeof(double)), "memset");
  if (s == GW_OK) s = launch_prologue(ctx, d_th, 1, 0, d_coef0, 1, nullptr, false);
  const TrigConsts T = make_trig_consts();
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_het_edges, dim3((ne + 255) / 256), dim3(256), 0, nullptr, ctx->bins, ctx->rec_stride,
                       d_edges, ne, nd, d_coef0, T, ctx->geom.k0, ctx->geom.df, h->rec);
    s = check_hip(hipGetLastError(), "het edge kernel");
  }
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_het_summary, dim3(ne - 1, nd), dim3(256), 0, nullptr, ctx->bins, ctx->rec_stride, d_hw, nf,
                       d_edges, ne - 1, d_coef0, T, ctx->geom.k0, ctx->geom.df, h->rec, nd);
    s = check_hip(hipGetLastError(), "het summary kernel");
  }
  double coef0[C_NCOEF];
  if (s == GW_OK) s = check_hip(hipMemcpy(coef0, d_coef0, sizeof(coef0), hipMemcpyDeviceToHost), "copy");
  if (s == GW_OK) s = check_hip(hipDeviceSynchronize(), "heterodyne set-up");
  cleanup();
  if (s != GW_OK) {
    free_state(h);
    return s;
  }
  for (int i = 0; i < nd; ++i) {
    const double ar = coef0[C_APRE + i], ai = coef0[C_APIM + i];
    const double m = ar * ar + ai * ai;
    if (!(m > 0.0)) {
      free_state(h);
      return set_error(GW_EINVAL, "heterodyne_setup: reference template vanishes in detector %d", i);
    }
    h->ap0_inv_re[i] = ar / m;
    h->ap0_inv_im[i] = -ai / m;
  }
  // Bin summaries -> per-edge weights of the summed-by-parts sums.
  {
    const int rs = h->rs, bo = het_bin_off(nd), nb = ne - 1;
    std::vector<double> rh((size_t)ne * rs);
    s = check_hip(hipMemcpy(rh.data(), h->rec, rh.size() * sizeof(double), hipMemcpyDeviceToHost), "copy");
    if (s != GW_OK) {
      free_state(h);
      return s;
    }
    std::vector<double> out(rh);
    for (int i = 0; i < nd; ++i) {
      double hh0 = 0.0;
      for (int e = 0; e < ne; ++e) {
        double rr = 0.0, ri = 0.0, lr = 0.0, li = 0.0, b0h = 0.0;
        if (e >= 1) {  // bin e: right edge e
          const double* sb = &rh[(size_t)e * rs + bo + 1 + 6 * i];
          const double inv = rh[(size_t)e * rs + bo];
          rr = 0.5 * sb[0] + sb[2] * inv;
          ri = 0.5 * sb[1] + sb[3] * inv;
          b0h = 0.5 * sb[4];
          hh0 += b0h;
        }
        if (e + 1 <= nb) {  // bin e + 1: left edge e
          const double* sb = &rh[(size_t)(e + 1) * rs + bo + 1 + 6 * i];
          const double inv = rh[(size_t)(e + 1) * rs + bo];
          lr = 0.5 * sb[0] - sb[2] * inv;
          li = 0.5 * sb[1] - sb[3] * inv;
        }
        double* o = &out[(size_t)e * rs + bo + 1 + 6 * i];
        o[0] = rr + lr;
        o[1] = ri + li;
        o[2] = rr;
        o[3] = ri;
        o[4] = b0h;
        o[5] = 0.0;
      }
      h->hh0[i] = hh0;
    }
    s = check_hip(hipMemcpy(h->rec, out.data(), out.size() * sizeof(double), hipMemcpyHostToDevice), "copy");
    if (s != GW_OK) {
      free_state(h);
      return s;
    }
  }
  ctx->het = h;
  ++ctx->gen;
  if (edges_out)
    for (int e = 0; e < ne; ++e) edges_out[e] = h->f_edges[e];
  return GW_OK;
}

gw_status gw_het_info(const gw_ctx* ctx, int32_t* n_bins) {
  if (!ctx || !n_bins) return set_error(GW_EINVAL, "gw_het_info: null argument");
  if (!ctx->het) return set_error(GW_ESTATE, "gw_het_info: heterodyne_setup has not been called");
  *n_bins = ctx->het->n_bins;
  return GW_OK;
}

gw_status loglike_batch_uneven(gw_ctx* ctx, const double* theta, int64_t n_rows, const int64_t* subs, int32_t n_sub,
                               int32_t like, int32_t marg, int32_t prec, int32_t use_graph, double* logl,
                               void* stream) {
  if (!ctx) return set_error(GW_EINVAL, "loglike_batch_uneven: ctx is NULL");
  if (n_rows < 0 || n_sub < 0) return set_error(GW_EINVAL, "loglike_batch_uneven: negative size");
  if (n_sub > kMaxSub) return set_error(GW_EINVAL, "loglike_batch_uneven: at most %d sub-batches", kMaxSub);
  if (n_sub > 0 && (!theta || !subs || !logl)) return set_error(GW_EINVAL, "loglike_batch_uneven: null pointer");
  if (like != GW_HET) return set_error(GW_ENOTSUP, "loglike_batch_uneven: only GW_HET is supported");
  if (marg < GW_MARG_NONE || marg > GW_MARG_PHASE_DIST) return set_error(GW_EINVAL, "loglike_batch_uneven: bad marg");
  if (prec != GW_PREC_FP64 && prec != GW_PREC_MIXED) return set_error(GW_EINVAL, "loglike_batch_uneven: bad prec");
  if (marg == GW_MARG_PHASE_DIST && ctx->n_dist <= 0)
    return set_error(GW_ESTATE, "loglike_batch_uneven: distance marginal needs a distance grid");
  if (!ctx->het) return set_error(GW_ESTATE, "loglike_batch_uneven: heterodyne_setup has not been called");
  if (n_sub == 0 || n_rows == 0) return GW_OK;
  hipStream_t st = (hipStream_t)stream;
  gw_status s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s != GW_OK) return s;
  gw_het_state* h = ctx->het;
  int n_ech = 1;
  s = het_prepare(ctx, theta, subs, n_sub, n_rows, logl, false, &n_ech, st);
  if (s != GW_OK) return s;
  if (!use_graph || ctx->prof) return enqueue_het(ctx, marg, prec, n_ech, st);

  if (!ctx->graphs) {
    ctx->graphs = new (std::nothrow) gw_graph_cache();
    if (!ctx->graphs) return set_error(GW_ENOMEM, "graph cache");
  }
  gw_graph_cache* gc = ctx->graphs;
  const GraphKey key{marg, prec, h->wpb, h->grid, n_ech, h->n_rows_last >= kDistRowsPerLane ? 1 : 0};
  auto it = gc->exec.find(key);
  if (it == gc->exec.end()) {
    if (!gc->cap_stream) {
      s = check_hip(hipStreamCreateWithFlags(&gc->cap_stream, hipStreamNonBlocking), "capture stream");
      if (s != GW_OK) return s;
    }
    hipGraph_t g = nullptr;
    hipGraphExec_t ge = nullptr;
    s = check_hip(hipStreamBeginCapture(gc->cap_stream, hipStreamCaptureModeThreadLocal), "begin capture");
    if (s != GW_OK) return s;
    gw_status sq = enqueue_het(ctx, marg, prec, n_ech, gc->cap_stream);
    s = check_hip(hipStreamEndCapture(gc->cap_stream, &g), "end capture");
    if (sq != GW_OK) {
      if (g) (void)hipGraphDestroy(g);
      return sq;
    }
    if (s != GW_OK) return s;
    const auto t0 = std::chrono::steady_clock::now();
    s = check_hip(hipGraphInstantiate(&ge, g, nullptr, nullptr, 0), "graph instantiate");
    const auto t1 = std::chrono::steady_clock::now();
    gc->last_instantiate_ms = std::chrono::duration<double, std::milli>(t1 - t0).count();
    if (s != GW_OK) {
      (void)hipGraphDestroy(g);
      return s;
    }
    gc->graph[key] = g;
    gc->exec[key] = ge;
    it = gc->exec.find(key);
  }
  return check_hip(hipGraphLaunch(it->second, st), "graph launch");
}

gw_status gw_set_het_shape(gw_ctx* ctx, int32_t waves_per_block, int32_t grid, int32_t n_ech) {
  if (!ctx) return set_error(GW_EINVAL, "gw_set_het_shape: ctx is NULL");
  if (!ctx->het) return set_error(GW_ESTATE, "gw_set_het_shape: heterodyne_setup has not been called");
  if (waves_per_block != 1 && waves_per_block != 2 && waves_per_block != 4)
    return set_error(GW_EINVAL, "gw_set_het_shape: waves_per_block must be 1, 2 or 4");
  if (grid < 0 || grid > (1 << 20)) return set_error(GW_EINVAL, "gw_set_het_shape: grid out of range");
  if (n_ech < 0 || n_ech > 256) return set_error(GW_EINVAL, "gw_set_het_shape: n_ech must be 0 .. 256");
  ctx->het->wpb = waves_per_block;
  ctx->het->grid = grid;
  ctx->het->ech = n_ech;
  ++ctx->gen;
  return GW_OK;
}

gw_status gw_set_het_tm_split(gw_ctx* ctx, int32_t n_chunks) {
  if (!ctx) return set_error(GW_EINVAL, "gw_set_het_tm_split: ctx is NULL");
  if (n_chunks < 0 || n_chunks > 256 || (n_chunks & (n_chunks - 1)) != 0)
    return set_error(GW_EINVAL, "gw_set_het_tm_split: n_chunks must be 0 or a power of two up to 256");
  ctx->tm_nsk = n_chunks;
  ++ctx->gen;
  return GW_OK;
}

gw_status gw_graph_info(const gw_ctx* ctx, int32_t* n_graphs, double* last_instantiate_ms) {
  if (!ctx || !n_graphs || !last_instantiate_ms) return set_error(GW_EINVAL, "gw_graph_info: null argument");
  *n_graphs = ctx->graphs ? (int32_t)ctx->graphs->exec.size() : 0;
  *last_instantiate_ms = ctx->graphs ? ctx->graphs->last_instantiate_ms : 0.0;
  return GW_OK;
}

// Autotuner: time every candidate launch shape on the caller's batch and keep
// the fastest in the context.  Candidates: full band, the automatic shape (the
// one in which a workgroup's waves share 64 rows) and proposals per workgroup
// {64, 128, 256} x frequency chunks {8 .. 512} (multiples of 8, at least 16
// bins per chunk); heterodyned, waves per workgroup {1, 2, 4} x persistent
// grid {8, 16, 32, 64} waves per CU x edge chunks {heuristic, 8, 16, 32}.
gw_status gw_autotune(gw_ctx* ctx, const double* theta, int64_t n, int32_t like, int32_t marg, int32_t prec,
                      int32_t reps, int32_t* best_shape, double* best_ms, void* stream) {
  if (!ctx || !theta || !best_shape || !best_ms) return set_error(GW_EINVAL, "gw_autotune: null argument");
  if (n < 1 || reps < 1) return set_error(GW_EINVAL, "gw_autotune: n and reps must be >= 1");
  if (like != GW_FULL && like != GW_HET) return set_error(GW_EINVAL, "gw_autotune: bad like");
  if (like == GW_HET && !ctx->het) return set_error(GW_ESTATE, "gw_autotune: heterodyne_setup has not been called");
  hipStream_t st = (hipStream_t)stream;
  gw_status s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s != GW_OK) return s;
  double* out = nullptr;
  s = check_hip(hipMalloc((void**)&out, (size_t)n * sizeof(double)), "autotune output");
  if (s != GW_OK) return s;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  const bool prof = ctx->prof;
  ctx->prof = false;
  struct Cand {
    int a, b, c;
  };
  std::vector<Cand> cands;
  if (like == GW_FULL) {
    cands.push_back({0, 0, 0});
    for (int tpb : {64, 128, 256})
      for (int ch : {8, 16, 32, 64, 128, 256, 512})
        if (ctx->geom.n_freq / ch >= 16) cands.push_back({tpb, ch, 0});
  } else {
    for (int w : {1, 2, 4})
      for (int per_cu : {8, 16, 32, 64})
        for (int ech : {0, 8, 16, 32}) cands.push_back({w, 256 * per_cu, ech});
  }
  double best = 1e300;
  Cand arg{0, 0, 0};
  for (const Cand& cand : cands) {
    if (like == GW_FULL) {
      ctx->full_tpb = cand.a;
      ctx->full_chunks = cand.b;
    } else {
      ctx->het->wpb = cand.a;
      ctx->het->grid = cand.b / cand.a;
      ctx->het->ech = cand.c;
    }
    s = loglike_batch(ctx, theta, n, like, marg, prec, out, st);  // warm-up
    if (s != GW_OK) break;
    (void)hipEventRecord(e0, st);
    for (int r = 0; r < reps && s == GW_OK; ++r) s = loglike_batch(ctx, theta, n, like, marg, prec, out, st);
    (void)hipEventRecord(e1, st);
    if (s != GW_OK) break;
    s = check_hip(hipEventSynchronize(e1), "autotune sync");
    if (s != GW_OK) break;
    float ms = 0.0f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    const double per = ms / reps;
    if (per < best) {
      best = per;
      arg = cand;
    }
  }
  if (like == GW_FULL) {
    ctx->full_tpb = arg.a;
    ctx->full_chunks = arg.b;
  } else {
    ctx->het->wpb = arg.a > 0 ? arg.a : 4;
    ctx->het->grid = arg.a > 0 ? arg.b / arg.a : 0;
    ctx->het->ech = arg.c;
    if (ctx->graphs) graphs_clear(ctx->graphs);
  }
  ctx->prof = prof;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipFree(out);
  if (s != GW_OK) return s;
  best_shape[0] = arg.a;
  best_shape[1] = like == GW_FULL ? arg.b : ctx->het->grid;
  best_shape[2] = arg.c;
  *best_ms = best;
  return GW_OK;
}

}  // extern "C"
