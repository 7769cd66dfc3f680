// Node tables of the full-band sums (gw_nodes.h): block partition on the host,
// interpolation weights on the device.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "gw_ctx.h"
#include "gw_nodes.h"
#include "gw_tgrid.h"

namespace gw {

// One node: its block's bins [kb, ke), the number of nodes n and its index j
// (n = ke - kb: a node per bin).
struct NodePlace {
  int32_t kb, ke, n, j;
};

// W_ij of one node and the reference phase at it (a workgroup per node, the
// block's bins over its threads, a fixed-order tree sum).  With the bins at
// f = f_c + h cos(theta) and the nodes at theta_j = (2 j + 1) pi / (2 n),
//   l_j = sin(theta_j) sin(n d) / (2 n sin((theta + theta_j) / 2) sin(d / 2)),
// d = theta - theta_j, which keeps its relative accuracy next to a node; theta
// comes from the bin's integer offset.  About 100 bins x nodes per bin, once
// per context: 1.1 ms at 259,585 bins.
__global__ void __launch_bounds__(256) k_node_weights(const NodePlace* __restrict__ place,
                                                      const double* __restrict__ bins, int nd, PhaseCoef ref,
                                                      TrigConsts T, int node_stride, double* __restrict__ rec) {
  const NodePlace P = place[blockIdx.x];
  const int rs = 4 + 2 * nd, nb = P.ke - P.kb;
  double acc[2 * kMaxDet];
#pragma unroll
  for (int i = 0; i < 2 * kMaxDet; ++i) acc[i] = 0.0;
  const double tj = (double)(2 * P.j + 1) * kPi / (double)(2 * P.n), sj = sin(tj);
  const int k0 = P.n == nb ? P.kb + P.j : P.kb, k1 = P.n == nb ? k0 + 1 : P.ke;
  for (int k = k0 + (int)threadIdx.x; k < k1; k += 256) {
    const double* __restrict__ b = bins + (int64_t)k * rs;
    double l = 1.0;
    if (P.n != nb) {
      // theta of the bin: cos(theta) = 1 - 2 q, q its distance from the top
      const int up = P.ke - 1 - k, dn = k - P.kb;
      const double inv = 1.0 / (double)(nb - 1);
      const double th = up <= dn ? 2.0 * asin(sqrt((double)up * inv)) : kPi - 2.0 * asin(sqrt((double)dn * inv));
      const double d = th - tj;
      if (d != 0.0)
        l = sj * sin((double)P.n * d) / (2.0 * P.n * sin(0.5 * (th + tj)) * sin(0.5 * d));
    }
    double s, c;
    sincos_cycles(phase_cycles(ref, b[0], b[1], b[2], b[3]), T, &s, &c);
    const double gr = l * c, gi = -l * s;
    for (int i = 0; i < nd; ++i) {
      const double ur = b[4 + 2 * i], ui = b[5 + 2 * i];
      acc[2 * i] += ur * gr - ui * gi;
      acc[2 * i + 1] += ur * gi + ui * gr;
    }
  }
  __shared__ double red[2 * kMaxDet][256];
#pragma unroll
  for (int i = 0; i < 2 * kMaxDet; ++i) red[i][threadIdx.x] = acc[i];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o)
      for (int i = 0; i < 2 * nd; ++i) red[i][threadIdx.x] += red[i][threadIdx.x + o];
    __syncthreads();
  }
  double* __restrict__ r = rec + (int64_t)blockIdx.x * node_stride;
  if ((int)threadIdx.x < 2 * nd) r[6 + threadIdx.x] = red[threadIdx.x][0];
  if (threadIdx.x == 0) r[5] = phase_cycles(ref, r[0], r[1], r[2], r[3]);
}

// Phase coefficients of the waveforms the tables are built for, by the rows'
// own prologue: the reference first, then the envelope's.
static gw_status node_waveforms(gw_ctx* ctx, std::vector<PhaseCoef>* out) {
  std::vector<double> th;
  auto put = [&](double mc, double q, double c1, double c2, double l1, double l2) {
    const double v[13] = {mc, q, c1, c2, l1, l2, 100.0, 0, 0, 0, 0, 0, 0};
    th.insert(th.end(), v, v + 13);
  };
  put(kNodeMc, 0.75, 0.0, 0.0, 0.0, 0.0);
  for (int m = 0; m < 64; ++m)
    put(m & 1 ? kNodeMc : 1.45, m & 2 ? 0.5 : 1.0, m & 4 ? 0.1 : -0.1, m & 8 ? 0.1 : -0.1, m & 16 ? 5000.0 : 0.0,
        m & 32 ? 5000.0 : 0.0);
  const int n = (int)(th.size() / 13);
  double* d = nullptr;
  gw_status s = check_hip(hipMalloc((void**)&d, (size_t)n * (13 + C_NCOEF) * sizeof(double)), "node waveforms");
  if (s != GW_OK) return s;
  std::vector<double> h((size_t)n * C_NCOEF);
  s = check_hip(hipMemcpy(d, th.data(), th.size() * sizeof(double), hipMemcpyHostToDevice), "node waveforms");
  if (s == GW_OK) s = launch_prologue(ctx, d, n, GW_MARG_PHASE_TIME, d + 13 * n, n, nullptr);
  if (s == GW_OK)
    s = check_hip(hipMemcpy(h.data(), d + 13 * n, h.size() * sizeof(double), hipMemcpyDeviceToHost), "node waveforms");
  (void)hipFree(d);
  if (s != GW_OK) return s;
  out->resize(n);
  for (int p = 0; p < n; ++p) {
    auto at = [&](int c) { return h[(size_t)c * n + p]; };
    (*out)[p] = PhaseCoef{at(C_A0), at(C_A2), at(C_A3), at(C_A4), at(C_A5), at(C_A6),
                          at(C_A7), 0.0,      at(C_A10), at(C_A12), at(C_B5), at(C_B6)};
  }
  PhaseCoef& r = (*out)[0];
  for (double* v : {&r.a0, &r.a2, &r.a3, &r.a4, &r.a5, &r.a6, &r.a7, &r.a10, &r.a12, &r.b5, &r.b6}) *v *= 0.5;
  return GW_OK;
}

// d Psi / d f on the host at x = f^(1/3) (phase_slope's terms).
static double slope_at(const PhaseCoef& c, double x, double lnf) {
  const double x2 = x * x, x3 = x2 * x;
  const double t = c.a0 * (-5.0 / 3.0) + x2 * (-c.a2 + x * (-2.0 / 3.0 * c.a3 + x * (-1.0 / 3.0 * c.a4 + x2 * (
      1.0 / 3.0 * c.a6 + x * (2.0 / 3.0 * c.a7 + x3 * (5.0 / 3.0 * c.a10 + x2 * 7.0 / 3.0 * c.a12))))));
  return t / (x3 * x3 * x2) + (c.b5 + c.b6 * x * (1.0 + lnf / 3.0)) / x3;
}

// Fewest nodes for omega radians to either side of the centre: one more than
// the smallest n > omega / 2 with 2 (omega / 2)^n / n! below the tolerance;
// kNodeMax + 1 for an omega beyond any block's.
struct NodeCount {
  double most[kNodeMax];  // largest omega of n = j + 1
  NodeCount() {
    for (int n = 1; n <= kNodeMax; ++n)
      most[n - 1] = 2.0 * fmin((double)n, exp((log(0.5 * kNodeTol) + lgamma(n + 1.0)) / n));
  }
  int operator()(double omega) const {
    if (!(omega < most[kNodeMax - 1])) return kNodeMax + 1;
    return (int)(std::upper_bound(most, most + kNodeMax, omega) - most) + 2;
  }
};

// S(f): the largest slope relative to the reference.
static double envelope(const std::vector<PhaseCoef>& w, double f) {
  const double x = cbrt(f), lnf = log(f), r = slope_at(w[0], x, lnf);
  double s = 0.0;
  for (size_t p = 1; p < w.size(); ++p) s = fmax(s, fabs(slope_at(w[p], x, lnf) - r));
  return 1.02 * s + 1e-3;
}

// S(f) by bin: the envelope on a grid fine enough for the larger of two
// neighbours to bound what lies between (power laws; 64 points an octave).
static void slope_bound(const Geom& g, const std::vector<PhaseCoef>& w, std::vector<double>* e) {
  const double k0 = (double)g.k0, f0 = k0 * g.df, top = (k0 + (double)(g.n_freq - 1)) / k0;
  const int n = 2 + (int)(64.0 * log2(top > 1.0 ? top : 1.0));
  e->resize(n + 1);
  for (int j = 0; j <= n; ++j) (*e)[j] = envelope(w, f0 * exp2(j / 64.0));
}

struct SlopeBound {
  const std::vector<double>& e;
  double k0;
  double at(int k) const {
    const int j = std::min((int)(64.0 * log2((k0 + k) / k0)), (int)e.size() - 2);
    return fmax(e[j], e[j + 1]);
  }
  // bins [k, l]: the envelope falls, then rises, so its ends bound a range
  double over(int k, int l) const { return fmax(at(k), at(l)); }
};

// Partition of the band: from the lowest bin up, the block length (growing by
// a quarter at a time, at most a sixth of its frequency, at most kNodeMax
// nodes) with the fewest nodes per bin.
static void partition(const gw_ctx* ctx, double tau, std::vector<NodePlace>* out) {
  const Geom& g = ctx->geom;
  const int nf = (int)g.n_freq;
  const NodeCount node_count;
  const SlopeBound slope{ctx->node_slope, (double)g.k0};
  for (int k = 0; k < nf;) {
    double best = 0.9;
    int bl = std::min(8, nf - k), bn = bl;  // a node per bin
    for (int L = 8; L <= nf - k; L = std::min(L + L / 4 + 1, L < nf - k ? nf - k : L + 1)) {
      const double f = (double)(g.k0 + k) * g.df, h = 0.5 * (L - 1) * g.df;
      if (L > 8 && 6.0 * L * g.df > f) break;
      const int n = node_count(kTwoPi * h * (slope.over(k, k + L - 1) + tau));
      if (n > kNodeMax) break;
      if ((double)n < best * L) {
        best = (double)n / L;
        bl = L;
        bn = n;
      }
    }
    for (int j = 0; j < bn; ++j) out->push_back(NodePlace{k, k + bl, bn, j});
    k += bl;
  }
}

// A node's offset from its block's first bin, in bins.
static double node_offset(const NodePlace& P) {
  if (P.n == P.ke - P.kb) return (double)P.j;
  return 0.5 * (double)(P.ke - 1 - P.kb) * (1.0 + cos((double)(2 * P.j + 1) * kPi / (double)(2 * P.n)));
}

// Records of the places, with ``extra`` further columns filled by the caller's
// ``fill(node, columns)``.
template <class Fill>
static gw_status node_table(gw_ctx* ctx, const PhaseCoef& ref, const std::vector<NodePlace>& place, int extra,
                            Fill fill, NodeTable* out) {
  const Geom& g = ctx->geom;
  const int nd = ctx->n_det, rs = node_rs(nd) + extra;
  const size_t n = place.size();
  std::vector<double> rec(std::max<size_t>(n, 1) * rs, 0.0);
  for (size_t q = 0; q < n; ++q) {
    const double f = ((double)(g.k0 + place[q].kb) + node_offset(place[q])) * g.df;
    double* r = &rec[q * rs];
    r[0] = cbrt(f);
    r[1] = r[0] * r[0];
    r[2] = pow(f, -5.0 / 3.0);
    r[3] = log(f);
    r[4] = f;
    fill(q, r + node_rs(nd));
  }
  // the places behind the records: one allocation and one copy
  static_assert(sizeof(NodePlace) == 2 * sizeof(double), "two columns a place");
  const size_t n_rec = rec.size();
  rec.resize(n_rec + 2 * n);
  if (n > 0) memcpy(&rec[n_rec], place.data(), n * sizeof(NodePlace));
  // published whole or not at all
  NodeTable t;
  gw_status s = check_hip(hipMalloc((void**)&t.rec, rec.size() * sizeof(double)), "node records");
  if (s == GW_OK) s = fault_tables("node records");
  if (s == GW_OK)
    s = check_hip(hipMemcpy(t.rec, rec.data(), rec.size() * sizeof(double), hipMemcpyHostToDevice), "records");
  if (s == GW_OK && n > 0) {
    hipLaunchKernelGGL(k_node_weights, dim3((unsigned)n), dim3(256), 0, nullptr, (const NodePlace*)(t.rec + n_rec),
                       (const double*)ctx->bins, nd, ref, make_trig_consts(), rs, t.rec);
    s = check_hip(hipGetLastError(), "node weights launch");
    if (s == GW_OK) s = check_hip(hipStreamSynchronize(nullptr), "node weights");
  }
  if (s != GW_OK) {
    if (t.rec) (void)hipFree(t.rec);
    return s;
  }
  t.n = (int)n;
  *out = t;
  return GW_OK;
}

static gw_status node_table(gw_ctx* ctx, const PhaseCoef& ref, const std::vector<NodePlace>& place, NodeTable* out) {
  return node_table(ctx, ref, place, 0, [](size_t, double*) {}, out);
}

// Largest light travel time from the geocentre to a detector.
static double travel_time(const Geom& g) {
  double rmax = 0.0;
  for (int i = 0; i < g.n_det; ++i)
    rmax = fmax(rmax, sqrt(g.pos[i][0] * g.pos[i][0] + g.pos[i][1] * g.pos[i][1] + g.pos[i][2] * g.pos[i][2]));
  return rmax / kLightSpeed;
}

gw_status nodes_init(gw_ctx* ctx) {
  std::vector<PhaseCoef> w;
  gw_status s = node_waveforms(ctx, &w);
  if (s != GW_OK) return s;
  const Geom& g = ctx->geom;
  NodeCheck& c = ctx->node_check;
  const double f0 = (double)g.k0 * g.df, f1 = (double)(g.k0 + g.n_freq - 1) * g.df;
  for (int j = 0; j < kNodeCheck; ++j) {
    const double f = f0 * pow(f1 / f0, (double)j / (kNodeCheck - 1)), x = cbrt(f);
    const double v[6] = {x, log(f), pow(x, -8.0), 1.0 / f, slope_at(w[0], x, log(f)), envelope(w, f)};
    memcpy(c.v[j], v, sizeof(v));
  }
  // the sampler's |t_c| <= 0.1 s prior at the geocentre or at any detector,
  // plus the light travel times; at most a quarter second
  c.tau_max = fmin(0.1 + 2.0 * travel_time(g), kTauCap);
  std::vector<NodePlace> place;
  slope_bound(g, w, &ctx->node_slope);
  ctx->node_ref = w[0];
  partition(ctx, c.tau_max, &place);
  s = check_hip(hipMalloc((void**)&ctx->node_check_dev, sizeof(NodeCheck)), "node check");
  if (s == GW_OK) s = check_hip(hipMemcpy(ctx->node_check_dev, &c, sizeof(c), hipMemcpyHostToDevice), "node check");
  if (s == GW_OK) s = node_table(ctx, ctx->node_ref, place, &ctx->nodes);
  return s;
}

gw_status nodes_wide_init(gw_ctx* ctx) {
  if (ctx->nodes_wide.rec) return GW_OK;
  std::vector<NodePlace> place;
  partition(ctx, kTauCap, &place);
  return node_table(ctx, ctx->node_ref, place, &ctx->nodes_wide);
}

// A wave's nodes, at least and at most, and the waves aimed at per 64 rows; a
// cell of more than twice its nodes is split over four waves.  Fewer per wave
// balance k_tspread better (1000 rows, 128 s: 72 us at 16, 75 at 48) but leave
// k_tgrid more chunks to add (86 us against 68): 147 us a call at 48, 149 at
// 32, 157 at 16; 50 to 1000 rows at 8 s are within 3 us either way.
constexpr int kTmNodesMin = 12, kTmNodesMax = 48, kTmWaves = 160;
// Most cells of a wave's nodes.
constexpr int kTmCells = 64;

// Tables of the time marginal: the nodes of the band for delays up to the
// window and the light travel time, each spread onto the grid at its own
// frequency, and their chunks.
gw_status tm_grid_init(gw_ctx* ctx, const TimeGridShape& g) {
  TmGrid& t = ctx->tm_grid;
  if (t.tab.rec && t.blk == g.blk && t.L == g.L && t.jmax == g.jmax) return GW_OK;
  tm_grid_free(ctx);
  const Geom& geom = ctx->geom;
  const int nf = (int)geom.n_freq, nd = ctx->n_det;
  std::vector<NodePlace> place;
  partition(ctx, (double)g.J * g.delta + travel_time(geom), &place);
  // Chebyshev nodes come from the top of their block down
  for (size_t q = 0; q < place.size();) {
    const size_t m = place[q].n;
    if (place[q].n != place[q].ke - place[q].kb) std::reverse(place.begin() + q, place.begin() + q + m);
    q += m;
  }
  const int n = (int)place.size(), n_cell = 2 * g.n_blk;
  std::vector<int32_t> cell(n);
  for (int q = 0; q < n; ++q)
    cell[q] = std::min((int)((place[q].kb + node_offset(place[q])) / g.cell), n_cell - 1);
  const int most = std::max(kTmNodesMin, std::min(kTmNodesMax, n / kTmWaves));
  const TgChunkPlan chunks = tgrid_chunks(cell, n_cell, most, kTmCells);
  const TgCoverPlan cn = tgrid_cover(chunks.a0, chunks.len, g.n_g);
  std::vector<int32_t> b0(g.n_blk), blen(g.n_blk, kTgW + 1);
  for (int b = 0; b < g.n_blk; ++b) b0[b] = 2 * b;
  const TgCoverPlan cb = tgrid_cover(b0, blen, g.n_g);
  const TgWindow win(g.beta);
  const int cell_bins = (g.blk + 1) / 2;
  std::vector<double> bw((size_t)cell_bins * kTgW);
  for (int k = 0; k < cell_bins; ++k) win.weights((double)k / g.cell, &bw[(size_t)k * kTgW]);
  // one allocation: the weights, then the integers, those read by fours first
  const int nc = chunks.n();
  std::vector<int32_t> idx;
  for (int c = 0; c < nc; ++c)
    for (const int32_t v : {chunks.first[c], chunks.first[c + 1], chunks.a0[c], cn.shift[c] + chunks.a0[c]})
      idx.push_back(v);
  size_t at[5];
  const std::vector<int32_t>* parts[5] = {&cn.pts, &cb.pts, &cell, &cn.shift, &cb.shift};
  for (int i = 0; i < 5; ++i) {
    at[i] = idx.size();
    idx.insert(idx.end(), parts[i]->begin(), parts[i]->end());
  }
  gw_status s = node_table(ctx, ctx->node_ref, place, kTgW, [&](size_t q, double* v) {
    win.weights((place[q].kb + node_offset(place[q])) / g.cell - cell[q], v);
  }, &t.tab);
  const size_t n_bw = bw.size();
  bw.resize(n_bw + (idx.size() + 1) / 2);
  memcpy(&bw[n_bw], idx.data(), idx.size() * sizeof(int32_t));
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&t.bins_w, bw.size() * sizeof(double)), "time-grid tables");
  if (s == GW_OK)
    s = check_hip(hipMemcpy(t.bins_w, bw.data(), bw.size() * sizeof(double), hipMemcpyHostToDevice), "tables");
  if (s != GW_OK) {
    tm_grid_free(ctx);
    return s;
  }
  t.idx = (const int32_t*)(t.bins_w + n_bw);
  t.chunk = (const int4*)t.idx;
  t.cell = t.idx + at[2];
  t.cov[0] = TgCover{(const int4*)(t.idx + at[0]), t.idx + at[3], cn.n_many};
  t.cov[1] = TgCover{(const int4*)(t.idx + at[1]), t.idx + at[4], cb.n_many};
  t.n_chunk = nc;
  t.n_dense = chunks.n_dense;
  t.n_pts = std::max(cn.n_pts, cb.n_pts);
  t.blk = g.blk;
  t.L = g.L;
  t.jmax = g.jmax;
  return GW_OK;
}

void tm_grid_free(gw_ctx* ctx) {
  TmGrid& t = ctx->tm_grid;
  if (t.tab.rec) (void)hipFree(t.tab.rec);
  if (t.bins_w) (void)hipFree(t.bins_w);
  t = TmGrid{};
}

void nodes_free(gw_ctx* ctx) {
  tm_grid_free(ctx);
  if (ctx->nodes_wide.rec) (void)hipFree(ctx->nodes_wide.rec);
  ctx->nodes_wide = NodeTable{};
  if (ctx->nodes.rec) (void)hipFree(ctx->nodes.rec);
  if (ctx->node_check_dev) (void)hipFree(ctx->node_check_dev);
  ctx->nodes = NodeTable{};
  ctx->node_check_dev = nullptr;
}

}  // namespace gw

extern "C" gw_status gw_full_nodes(const gw_ctx* ctx, int32_t* n_nodes, double* tau_max) {
  if (!ctx) return gw::set_error(GW_EINVAL, "gw_full_nodes: ctx is NULL");
  if (n_nodes) *n_nodes = ctx->nodes.n;
  if (tau_max) *tau_max = ctx->node_check.tau_max;
  return GW_OK;
}
