// Coalescence-time marginal on the full band (Sec. III.A and the appendix on
// grid marginalisations: a log-sum-exp over a grid of time shifts, computed
// by FFT on the uniform grid), together with the phase marginal.
//
// Grid: t_j = j delta, |j| <= J = floor(W / delta), delta = 1 / (N df) with N
// the smallest power of two >= 2 (k0 + n_freq - 1) (the segment's sampling
// interval).  With the template at t_c = 0,
//   log L = -<d|d>/2 - <h|h>/2 + ln[ (1 / (2J + 1)) sum_j I0(|Z(t_j)|) ],
//   Z(t)  = sum_k y_k exp(-2 pi i f_k t),
//   y_k   = 4 df sum_i d_ik* h_ik / S_ik = g_k sum_i (A P_i) u_ik exp(-2 pi i f_k dtau_i),
// g_k the detector-0 phasor (template phase including detector 0's delay) and
// dtau_i the other detectors' delays relative to detector 0.
//
// Evaluation.  The samples y are spread onto a coarse frequency grid and one
// transform of that grid gives every Z(t_j) (gw_tgrid.hip):
//   k_tspread, k_tbins: per proposal, the grid sums in chunks (lane =
//              proposal, wave-uniform records), from interpolation nodes or
//              from the bins of proposals outside the node tables;
//   k_tgrid:   one workgroup per proposal, transform, ln I0(|Z|) and a
//              fixed-order log-sum-exp.
// Rows go through in chunks whose grid sums fit a bounded workspace.
#include <math.h>

#include <vector>

#include "gw_ctx.h"
#include "gw_phase.h"
#include "gw_tgrid.h"

namespace gw {

constexpr int kTMaxP = 2048;

template <int PREC>
__device__ inline void tm_phasor(double r, const TrigConsts& T, double* gr, double* gi) {
  if (PREC == 0) {
    double s, c;
    sincos_cycles(r, T, &s, &c);
    *gr = c;
    *gi = -s;
  } else {
    const float t = (float)(r - rint(r));
    *gr = (double)__builtin_amdgcn_cosf(t);
    *gi = -(double)__builtin_amdgcn_sinf(t);
  }
}

// The phase coefficients of one row.
__device__ inline PhaseCoef tm_phase_coef(const double* __restrict__ coef, int64_t ld, int64_t pc) {
  PhaseCoef c;
  c.a0 = coef[C_A0 * ld + pc];
  c.a2 = coef[C_A2 * ld + pc];
  c.a3 = coef[C_A3 * ld + pc];
  c.a4 = coef[C_A4 * ld + pc];
  c.a5 = coef[C_A5 * ld + pc];
  c.a6 = coef[C_A6 * ld + pc];
  c.a7 = coef[C_A7 * ld + pc];
  c.a8 = coef[C_A8 * ld + pc];
  c.a10 = coef[C_A10 * ld + pc];
  c.a12 = coef[C_A12 * ld + pc];
  c.b5 = coef[C_B5 * ld + pc];
  c.b6 = coef[C_B6 * ld + pc];
  return c;
}

// Rows that the node tables cover (gw_nodes.h; delays here are at most the
// light travel time).  Lane = row, a workgroup of four waves per (64-row tile,
// unit): the first n_dense units are a cell each, whose nodes the four waves
// share (their sums added in a fixed order), the others four chunks of cells, a
// wave each, whose window of kTgW grid points slides: a point that no later
// node reaches is stored.
//
// Measured at 1000 rows, 128 s, 20-2048 Hz, three detectors, mixed: 808 us for
// twelve Chebyshev moments of every 512 bins, 120 us for these over nodes,
// 76 us here (6,880 nodes, 133 vector operations each: 24 us at full rate; 40
// MB written).  Bound by latency and by the uneven fill of 624 workgroups on
// 256 CUs.  The tiles of a unit go to the XCDs in turn: all units of a tile on
// one XCD, whose L2 would merge their 16-byte stores, takes 92 us a call
// against 71 at 250 rows (four XCDs busy), 147 both at 1000.
template <int ND, int PREC>
__global__ void __launch_bounds__(256, 4) k_tspread(const double* __restrict__ coef, int64_t ld, int64_t n,
                                                    TrigConsts T, TrigFit F, const double* __restrict__ nodes,
                                                    const int32_t* __restrict__ cells,
                                                    const int4* __restrict__ chunks, int n_chunk, int n_dense,
                                                    int64_t pitch, double2* __restrict__ part) {
  constexpr int NB = node_rs(ND), NS = NB + kTgW;
  __shared__ double red[2][2 * kTgW][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nptile = (int)((n + 63) / 64);
  const int unit = blockIdx.x / nptile, ptile = blockIdx.x - unit * nptile;
  const int64_t p = (int64_t)ptile * 64 + lane;
  const int64_t pc = p < n ? p : n - 1;
  const bool mine = p < n && coef[C_NODE * ld + pc] >= kNodePhase;
  if (__ballot(mine) == 0) return;  // the same in the workgroup's four waves
  double2* __restrict__ row = part + p * pitch;
  const PhaseCoef c = tm_phase_coef(coef, ld, pc);
  const bool dense = unit < n_dense;
  const int ch = dense ? unit : n_dense + 4 * (unit - n_dense) + wv;
  if (ch >= n_chunk) return;
  const int4 C = chunks[ch];
  int jb = C.x, je = C.y;
  if (dense) {
    const int nsub = (je - jb + 3) / 4;
    jb = jb + wv * nsub < je ? jb + wv * nsub : je;
    je = jb + nsub < je ? jb + nsub : je;
  }
  double mr[kTgW], mi[kTgW];
#pragma unroll
  for (int m = 0; m < kTgW; ++m) mr[m] = mi[m] = 0.0;
  double2* out = row + C.w;
  int cur = C.z;
  double qr[ND], qi[ND], dt[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    qr[i] = coef[(C_APRE + i) * ld + pc];
    qi[i] = coef[(C_APIM + i) * ld + pc];
    dt[i] = i == 0 ? 0.0 : coef[(C_DT1 + i - 1) * ld + pc];
  }
  auto step = [&](const double* __restrict__ rec, int j) {
    const double* __restrict__ w = nodes + (int64_t)j * NS + NB;
    const int cell = cells[j];
    const double r0 = node_phase(c, rec[0], rec[1], rec[2], rec[3], rec[5]);
    double yr = 0.0, yi = 0.0;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      double gr, gi;
      node_phasor<PREC>(i == 0 ? r0 : fma(rec[4], dt[i], r0), T, F, &gr, &gi);
      const double ur = rec[6 + 2 * i], ui = rec[7 + 2 * i];
      const double wr = fma(ur, gr, -ui * gi), wi = fma(ur, gi, ui * gr);
      yr = fma(qr[i], wr, fma(-qi[i], wi, yr));
      yi = fma(qr[i], wi, fma(qi[i], wr, yi));
    }
    for (; cur < cell; ++cur, ++out) {
      if (mine) *out = make_double2(mr[0], mi[0]);
#pragma unroll
      for (int m = 0; m + 1 < kTgW; ++m) {
        mr[m] = mr[m + 1];
        mi[m] = mi[m + 1];
      }
      mr[kTgW - 1] = mi[kTgW - 1] = 0.0;
    }
#pragma unroll
    for (int m = 0; m < kTgW; ++m) {
      mr[m] = fma(w[m], yr, mr[m]);
      mi[m] = fma(w[m], yi, mi[m]);
    }
  };
  if (je > jb) {  // in pairs, the next record in flight
    double ra[NB], rb[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) ra[q] = nodes[(int64_t)jb * NS + q];
    int j = jb;
    for (; j + 2 <= je; j += 2) {
#pragma unroll
      for (int q = 0; q < NB; ++q) rb[q] = nodes[(int64_t)(j + 1) * NS + q];
      step(ra, j);
      const int j2 = j + 2 < je ? j + 2 : je - 1;
#pragma unroll
      for (int q = 0; q < NB; ++q) ra[q] = nodes[(int64_t)j2 * NS + q];
      step(rb, j + 1);
    }
    if (j < je) step(ra, j);
  }
  if (dense) {  // (0 + 2) + (1 + 3)
    auto put = [&](int at) {
#pragma unroll
      for (int m = 0; m < kTgW; ++m) {
        red[at][2 * m][lane] = mr[m];
        red[at][2 * m + 1][lane] = mi[m];
      }
    };
    auto take = [&](int at) {
#pragma unroll
      for (int m = 0; m < kTgW; ++m) {
        mr[m] += red[at][2 * m][lane];
        mi[m] += red[at][2 * m + 1][lane];
      }
    };
    if (wv >= 2) put(wv - 2);
    __syncthreads();
    if (wv < 2) take(wv);
    __syncthreads();
    if (wv == 1) put(0);
    __syncthreads();
    if (wv > 0) return;
    take(0);
  }
  if (mine) {
#pragma unroll
    for (int m = 0; m < kTgW; ++m) out[m] = make_double2(mr[m], mi[m]);
  }
}

// The other rows (all: every row), over the bins.  Lane = row, the tiles by kind of
// row (tile_row).  A wave takes a block's upper cell, then its lower one, adding the
// upper one's points to it from memory, or, in a launch of few waves (PAIR), two
// waves a cell each, the lower one's adding the upper one's from LDS: the same sums
// (64 rows of 128 s, mixed: 439 us a call in one wave, 239 in two).  A tile with no
// such row leaves at once (5 us for 16 tiles of 128 s, 8 in pairs).  A kernel of its
// own: in one launch with the nodes, parted by workgroup, both spill (1000 rows within
// the tables: 290 us a call against 148).  The cell's bins are walked from the top
// down (wave-uniform records).  FP64: the phase of every bin by its full series.
// Mixed: the phase by the cubic recurrence in the runs of the full-band walk
// (gw_phase.h: a bin's phase depends on its run alone, so it is the same here as in
// the distance-marginal reduction), FP32 hardware sin/cos, FP64 sums.
// e_i = (A P_i) exp(-2 pi i f_k dtau_i) starts at the cell's top bin and
// steps down by conj(rho_i), rho_i = exp(-2 pi i df dtau_i).
template <int ND, int PREC, bool PAIR>
__global__ void __launch_bounds__(256, 4) k_tbins(const double* __restrict__ coef, int64_t ld, int64_t n, bool all,
                                                  const double* __restrict__ bins, int64_t k0, double df, int n_freq,
                                                  int blk, int n_blk, TrigConsts T, PhaseRuns R, double pg_re,
                                                  double pg_im, const double* __restrict__ basis, int64_t pitch,
                                                  double2* __restrict__ part) {
  constexpr int RS = 4 + 2 * ND;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the tiles of a unit are rotated by the unit: those without such a row leave, and
  // the rest then fall on all XCDs and on all of an XCD's engines, to which
  // workgroups are dealt in turn (500 of 1000 rows of 128 s: 946 us with every second
  // workgroup of an XCD one that leaves, 1030 for all rows)
  const int nptile = (int)((n + 63) / 64);
  const int unit = blockIdx.x / nptile;
  int ptile = blockIdx.x - unit * nptile + ((unit + (unit >> 2)) & 15);
  while (ptile >= nptile) ptile -= nptile;
  const TileRow r = all ? TileRow{(int64_t)ptile * 64 + lane, false} : tile_row(coef, ld, n, ptile, lane);
  const int64_t p = r.p, pc = p < n ? p : n - 1;
  const bool mine = p < n && !r.covered;
  if (!__any(mine)) return;
  const PhaseCoef c = tm_phase_coef(coef, ld, pc);
  constexpr int K = kTgW;
  const int b = PAIR ? 2 * unit + (wv >> 1) : 4 * unit + wv;
  const int b0 = b * blk, b1 = b0 + blk < n_freq ? b0 + blk : n_freq, mid = b0 + (blk + 1) / 2;
  int kb = 0, ke = 0;  // the cell's bins
  double mr[K], mi[K];
  double er[ND], ei[ND], rr[ND], ri[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    rr[i] = 1.0;
    ri[i] = 0.0;
    if (i > 0) {
      double s, co;
      sincos_cycles(df * coef[(C_DT1 + i - 1) * ld + pc], T, &s, &co);
      rr[i] = co;
      ri[i] = s;  // conj(rho_i): the walk descends
    }
  }
  // one bin: y = g sum_i u_ik e_i into the moments, then e_i one bin down
  auto visit = [&](int k, double gr, double gi) {
    const double* __restrict__ u = bins + (int64_t)k * RS + 4;
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const double ur = u[2 * i], ui = u[2 * i + 1];
      sr = fma(ur, er[i], sr);
      sr = fma(-ui, ei[i], sr);
      si = fma(ur, ei[i], si);
      si = fma(ui, er[i], si);
      if (i > 0) {
        const double tr = er[i] * rr[i] - ei[i] * ri[i];
        ei[i] = er[i] * ri[i] + ei[i] * rr[i];
        er[i] = tr;
      }
    }
    const double yr = gr * sr - gi * si, yi = gr * si + gi * sr;
    // the grid weights of the bin's offset in its cell (the same for every
    // cell and proposal: wave-uniform scalar loads)
    const double* __restrict__ tq = basis + (int64_t)(k - kb) * K;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      mr[m] = fma(tq[m], yr, mr[m]);
      mi[m] = fma(tq[m], yi, mi[m]);
    }
  };
  auto cell = [&](bool upper) {
    kb = upper ? mid : b0;
    ke = upper ? b1 : (b1 < mid ? b1 : mid);  // no bins beyond the band
#pragma unroll
    for (int m = 0; m < K; ++m) mr[m] = mi[m] = 0.0;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const double apr = coef[(C_APRE + i) * ld + pc], api = coef[(C_APIM + i) * ld + pc];
      er[i] = apr;
      ei[i] = api;
      if (i > 0) {
        double s, co;
        sincos_cycles((double)(k0 + ke - 1) * df * coef[(C_DT1 + i - 1) * ld + pc], T, &s, &co);
        er[i] = apr * co + api * s;
        ei[i] = api * co - apr * s;
      }
    }
    if constexpr (PREC == 0) {
      for (int k = ke - 1; k >= kb; --k) {
        const double* __restrict__ rec = bins + (int64_t)k * RS;
        double gr, gi;
        tm_phasor<0>(phase_cycles(c, rec[0], rec[1], rec[2], rec[3]), T, &gr, &gi);
        visit(k, gr, gi);
      }
    } else {
      // One run at a time: its top (up to) four bins evaluated directly give
      // the backward differences; every bin of the run in this block is then
      // visited from one call site (direct phases for the top bins, the
      // recurrence below them), which keeps the loop body small.  A block
      // that starts inside a run advances the recurrence through the run's
      // bins above it without visiting them.
      const double lin_step = -c.a8 * df;  // linear phase change per bin of the descending walk
      int k = ke - 1;
      while (k >= kb) {
        int L = 0, s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int sj = k & ~(R.len[j] - 1);
          if (L == 0 && sj >= R.k_min[j]) {
            L = R.len[j];
            s = sj;
          }
        }
        // a bin below the lowest level is a run of one, evaluated directly
        const int top = L == 0 ? k : (s + L - 1 < n_freq - 1 ? s + L - 1 : n_freq - 1);
        if (L == 0) s = k;
        const int nd = top - s + 1 < 4 ? top - s + 1 : 4;
        double r0 = 0.0, r1 = 0.0, r2 = 0.0, r3 = 0.0;  // direct phases of bins top, top - 1, ...
        double n0 = 0.0, n1 = 0.0, n2 = 0.0, n3 = 0.0, lin = 0.0;
#pragma nounroll
        for (int j = 0; j < nd; ++j) {
          const double* __restrict__ rc = bins + (int64_t)(top - j) * RS;
          const double nl = phase_nonlinear(c, rc[0], rc[1], rc[2], rc[3]);
          lin = fma(c.a8, rc[0] * rc[1], c.a5);
          const double d1 = nl - n0;
          const double d2 = d1 - n1;
          n3 = d2 - n2;
          n2 = d2;
          n1 = d1;
          n0 = nl;
          const double ph = nl + lin;
          r0 = j == 0 ? ph : r0;
          r1 = j == 1 ? ph : r1;
          r2 = j == 2 ? ph : r2;
          r3 = j == 3 ? ph : r3;
        }
        double p0 = n0 + lin, p1 = n1 + lin_step, p2 = n2;
        const double p3 = n3;
        int kk = top - nd;
        for (; kk > k; --kk) {  // above the walk's first bin: advance only
          p2 += p3;
          p1 += p2;
          p0 += p1;
        }
        const int lo = s > kb ? s : kb;
        for (kk = k; kk >= lo; --kk) {
          const int j = top - kk;
          double ph;
          if (j < nd) {
            ph = j == 0 ? r0 : (j == 1 ? r1 : (j == 2 ? r2 : r3));
          } else {
            p2 += p3;
            p1 += p2;
            p0 += p1;
            ph = p0;
          }
          double gr, gi;
          tm_phasor<1>(ph, T, &gr, &gi);
          visit(kk, gr, gi);
        }
        k = s - 1;
      }
    }
    if (PREC == 1) {  // remove the mean bias of the hardware phasor
#pragma unroll
      for (int m = 0; m < K; ++m) {
        const double tr = mr[m] * pg_re - mi[m] * pg_im;
        mi[m] = mr[m] * pg_im + mi[m] * pg_re;
        mr[m] = tr;
      }
    }
  };
  if constexpr (PAIR) {
    __shared__ double red[2][2 * K][64];
    const bool upper = wv & 1;
    cell(upper);
    if (upper) {
#pragma unroll
      for (int m = 0; m < K; ++m) {
        red[wv >> 1][2 * m][lane] = mr[m];
        red[wv >> 1][2 * m + 1][lane] = mi[m];
      }
    }
    __syncthreads();
    if (upper || !mine || b >= n_blk) return;
    double2* __restrict__ out = part + p * pitch + (int64_t)b * (K + 1);
    const double (*hi)[64] = red[wv >> 1];
    out[0] = make_double2(mr[0], mi[0]);
#pragma unroll
    for (int m = 1; m < K; ++m)
      out[m] = make_double2(mr[m] + hi[2 * m - 2][lane], mi[m] + hi[2 * m - 1][lane]);
    out[K] = make_double2(hi[2 * K - 2][lane], hi[2 * K - 1][lane]);
  } else {
    if (b >= n_blk) return;
    double2* out = part + p * pitch + (int64_t)b * (K + 1);
#pragma nounroll
    for (int upper = 1; upper >= 0; --upper) {
      cell(upper);
      if (!mine) continue;
      if (upper) {
#pragma unroll
        for (int m = 0; m < K; ++m) out[m + 1] = make_double2(mr[m], mi[m]);
      } else {
        out[0] = make_double2(mr[0], mi[0]);
#pragma unroll
        for (int m = 1; m < K; ++m) {
          const double2 hi = out[m];
          out[m] = make_double2(mr[m] + hi.x, mi[m] + hi.y);
        }
      }
    }
  }
}

template <int ND>
static void launch_tspread(gw_ctx* ctx, const double* coef, int64_t ld, int64_t n, int prec, int blk, int n_blk,
                           double2* part, hipStream_t st) {
  const TmGrid& t = ctx->tm_grid;
  const int64_t nptile = (n + 63) / 64;
  const bool fp64 = prec == GW_PREC_FP64, nodes = ctx->full_kernel != 1;
  if (nodes) {
    const int n_units = t.n_dense + (t.n_chunk - t.n_dense + 3) / 4;
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)(nptile * n_units)), dim3(256), 0, st, coef, ld, n,
                         make_trig_consts(), make_trig_fit(), (const double*)t.tab.rec, t.cell, t.chunk, t.n_chunk,
                         t.n_dense, (int64_t)t.n_pts, part);
    };
    fp64 ? launch(k_tspread<ND, 0>) : launch(k_tspread<ND, 1>);
  }
  // in pairs while the waves then still run all at once (four a SIMD)
  const bool pair = nptile * 2 * n_blk <= 4096;
  auto launch = [&](auto kernel) {
    const int units = pair ? (n_blk + 1) / 2 : (n_blk + 3) / 4;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(nptile * units)), dim3(256), 0, st, coef, ld, n, !nodes, ctx->bins,
                       ctx->geom.k0, ctx->geom.df, (int)ctx->geom.n_freq, blk, n_blk, make_trig_consts(),
                       make_phase_runs(ctx->geom), fp64 ? 1.0 : ctx->pgain_re, fp64 ? 0.0 : ctx->pgain_im,
                       (const double*)t.bins_w, (int64_t)t.n_pts, part);
  };
  if (pair)
    fp64 ? launch(k_tbins<ND, 0, true>) : launch(k_tbins<ND, 1, true>);
  else
    fp64 ? launch(k_tbins<ND, 0, false>) : launch(k_tbins<ND, 1, false>);
}

gw_status time_grid_shape(const gw_ctx* ctx, TimeGridShape* g) {
  const int64_t top = 2 * (ctx->geom.k0 + ctx->geom.n_freq - 1);
  int64_t N = 1;
  while (N < top) N <<= 1;
  g->N = N;
  g->delta = 1.0 / ((double)N * ctx->geom.df);
  g->J = (int)floor(ctx->tm_window / g->delta + 1e-9);
  g->R = ctx->tm_R;
  // P >= 2 J + 1, and at least 16 / R so that the transform has 16 points
  int P = 2;
  while (P < 2 * g->J + 1 || P * g->R < 16) P <<= 1;
  if (P > kTMaxP) return set_error(GW_ENOTSUP, "time marginal: window %.6g s needs more than %d grid points",
                                   ctx->tm_window, kTMaxP);
  if (N / P < 1) return set_error(GW_ENOTSUP, "time marginal: grid finer than the segment's sampling");
  g->P = P;
  g->blk = (int)(N / P);
  g->n_blk = (int)((ctx->geom.n_freq + g->blk - 1) / g->blk);
  g->L = P * g->R;
  g->jmax = g->J * g->R;
  int D1, D2;
  if (!tgrid_plan(g->L, &D1, &D2))
    return set_error(GW_ENOTSUP, "time marginal: %d grid points per sampling interval over +-%.6g s need a "
                                 "%d-point transform (at most 4096)", g->R, ctx->tm_window, g->L);
  g->cell = 0.5 * g->blk;
  g->n_g = 2 * g->n_blk + kTgW - 1;
  g->beta = tgrid_beta((double)g->jmax / (2.0 * g->L));
  g->f0_num = (double)ctx->geom.k0 - kTgLead * g->cell;
  g->f0_den = (double)g->N * (double)g->R;
  return GW_OK;
}

gw_status loglike_tmarg(gw_ctx* ctx, const double* theta, int64_t n, int prec, double* logl, hipStream_t st) {
  return loglike_tmarg_staged(ctx, theta, n, prec, logl, nullptr, st);
}

gw_status loglike_tmarg_staged(gw_ctx* ctx, const double* theta, int64_t n, int prec, double* logl, double* zout,
                               hipStream_t st) {
  TimeGridShape g;
  gw_status s = time_grid_shape(ctx, &g);
  if (s == GW_OK) s = tgrid_tables(ctx, g.L, g.jmax);
  if (s == GW_OK) s = tm_grid_init(ctx, g);
  if (s != GW_OK) return s;
  const TmGrid& t = ctx->tm_grid;
  // whole groups of tiles (tile_row)
  constexpr int64_t kGroup = 64 * kTileGroup;
  int64_t chunk = tgrid_chunk_rows(n, t.n_pts);
  if (chunk < n) chunk = chunk > kGroup ? chunk / kGroup * kGroup : kGroup;
  const int nt = 2 * g.jmax + 1;
  s = ensure_buffer(&ctx->coef, &ctx->coef_cap, (int64_t)C_NCOEF * n, "coefficient workspace");
  if (s == GW_OK) s = ensure_buffer(&ctx->tm_mom, &ctx->tm_mom_cap, chunk * t.n_pts * 2, "time-grid sums");
  if (s != GW_OK || !theta) return s;  // theta NULL: reserve only
  s = launch_prologue(ctx, theta, n, GW_MARG_PHASE_TIME, ctx->coef, n, st);
  if (s != GW_OK) return s;
  double2* part = (double2*)ctx->tm_mom;
  for (int64_t r0 = 0; r0 < n && s == GW_OK; r0 += chunk) {
    const int64_t cn = n - r0 < chunk ? n - r0 : chunk;
    const int slot = prof_begin(ctx, st, 1);
    switch (ctx->n_det) {
      case 1: launch_tspread<1>(ctx, ctx->coef + r0, n, cn, prec, g.blk, g.n_blk, part, st); break;
      case 2: launch_tspread<2>(ctx, ctx->coef + r0, n, cn, prec, g.blk, g.n_blk, part, st); break;
      case 3: launch_tspread<3>(ctx, ctx->coef + r0, n, cn, prec, g.blk, g.n_blk, part, st); break;
      case 4: launch_tspread<4>(ctx, ctx->coef + r0, n, cn, prec, g.blk, g.n_blk, part, st); break;
      default: return set_error(GW_ENOTSUP, "n_det %d not supported", ctx->n_det);
    }
    prof_end(ctx, slot, st);
    s = check_hip(hipGetLastError(), "time-grid sums launch");
    if (s != GW_OK) return s;
    TGridArgs a{};
    a.part = ctx->tm_mom;
    a.pitch = t.n_pts;
    a.cov[0] = t.cov[0];
    a.cov[1] = t.cov[1];
    a.node_from = ctx->full_kernel != 1 ? kNodePhase : INFINITY;
    a.n = cn;
    a.n_g = g.n_g;
    a.L = g.L;
    a.jmax = g.jmax;
    a.coef = ctx->coef + r0;
    a.ld = n;
    a.logl = logl + r0;
    a.zout = zout ? zout + r0 * nt * 3 : nullptr;
    a.f0_num = g.f0_num;
    a.f0_den = g.f0_den;
    const int gslot = prof_begin(ctx, st, 2);
    s = launch_tgrid(ctx, a, st);
    prof_end(ctx, gslot, st);
  }
  return s;
}

gw_status tmarg_reserve(gw_ctx* ctx, int64_t n, int like) {
  return like == GW_HET ? loglike_het_tmarg_staged(ctx, nullptr, n, GW_PREC_FP64, nullptr, nullptr, 0)
                        : loglike_tmarg_staged(ctx, nullptr, n, GW_PREC_FP64, nullptr, nullptr, 0);
}

}  // namespace gw

extern "C" gw_status gw_set_time_window(gw_ctx* ctx, double window) {
  if (!ctx) return gw::set_error(GW_EINVAL, "gw_set_time_window: ctx is NULL");
  if (!(window >= 0.0) || !isfinite(window)) return gw::set_error(GW_EINVAL, "gw_set_time_window: window >= 0");
  const double old = ctx->tm_window;
  ctx->tm_window = window;
  gw::TimeGridShape g;
  const gw_status s = gw::time_grid_shape(ctx, &g);
  if (s != GW_OK) ctx->tm_window = old;
  else ++ctx->gen;
  return s;
}

extern "C" gw_status gw_set_time_oversample(gw_ctx* ctx, int32_t factor) {
  if (!ctx) return gw::set_error(GW_EINVAL, "gw_set_time_oversample: ctx is NULL");
  if (factor != 1 && factor != 2 && factor != 4 && factor != 8 && factor != 16)
    return gw::set_error(GW_EINVAL, "gw_set_time_oversample: factor must be 1, 2, 4, 8 or 16");
  ctx->tm_R = factor;
  ++ctx->gen;
  return GW_OK;
}

extern "C" gw_status gw_time_grid_info(const gw_ctx* ctx, double* delta, int32_t* n_points, int32_t* fft_len,
                                       int32_t* block_bins) {
  if (!ctx) return gw::set_error(GW_EINVAL, "gw_time_grid_info: ctx is NULL");
  gw::TimeGridShape g;
  const gw_status s = gw::time_grid_shape(ctx, &g);
  if (s != GW_OK) return s;
  if (delta) *delta = g.delta / g.R;
  if (n_points) *n_points = 2 * g.J * g.R + 1;
  if (fft_len) *fft_len = g.P;
  if (block_bins) *block_bins = g.blk;
  return GW_OK;
}
