// Grid sum over coalescence-time shifts (Sec. III.A and the appendix on grid
// marginalisations), shared by the full-band and heterodyned time marginals.
//
// The shifts are t_j = j delta / R, |j| <= jmax = J R, with delta the
// segment's sampling interval 1 / (N df), and
//   Z(t_j) = sum_k y_k exp(-2 pi i f_k t_j)
// over samples y_k at frequencies f_k (interpolation nodes or bins of the full
// band, edges of the heterodyned bins).  The samples are spread onto a uniform
// frequency grid of cells of N / (2 P) bins (P a power of two >= 2 J + 1) with
// a Kaiser-Bessel window of kTgW points (gw_tgrid.h), G_g = sum_k y_k
// psi(x_k - g), x_k = f_k / cell; then
//   Z(t_j) = exp(-2 pi i f_0 t_j) / psi_hat(nu_j) sum_g G_g exp(-2 pi i g nu_j),
// nu_j = j / (2 L), L = P R, |nu_j| < 1/4: one transform of 2 L points, taken as
// its even (r = 0) and odd (r = 1) outputs j = 2 j' + r, each a transform of L
// points of G_g exp(-2 pi i g r / (2 L)) with the points g >= L folded onto
// g - L (sign (-1)^r).  The window's images stay below 6e-13 of sum |y|
// (5e-14 at the default window).  exp(-2 pi i f_0 t_j), f_0 the frequency of
// g = 0, has unit modulus.
//
// The kernels that form the y_k leave G in chunks: chunk c holds the sums of
// its samples over the grid points they reach, and neighbouring chunks overlap
// (tgrid_cover); k_tgrid adds the chunks of each point in order.
//
// k_tgrid: 256 lanes per row and r.  An in-place decimation-in-frequency FFT of
// L = D1 D2 16 points (D1 = L / 256 for L >= 256, else D1 = 1 and D2 = L / 16)
// in three passes: the first on the lane's grid points in registers (points at
// or beyond n_g are zero; for L = 4096 the radix-16 butterfly skips the inputs
// known to be zero), the second in LDS, and the third leaves each lane its 16
// outputs.  The LDS buffer stores element i at i + floor(i / 16), which keeps
// all three access patterns free of bank conflicts.  Twiddles are powers of one
// root of unity per lane, formed by repeated products.  Then ln I0(|Z|) -
// <h|h>(t_j) / 2 and a fixed-order log-sum-exp.  For the heterodyned bins the
// norm also depends on t_j:
// <h|h>(t_j) = hhc + Re exp(-2 pi i c u_j) sum_{m < MH} (-i x_j)^m / m! S_m,
// u_j = j / (N R) (fine-grid cycles), x_j = 2 pi hw u_j, with the bin widths
// dk_e = c + hw sigma_e expanded about their centre c and S_m the per-row
// moments sum_e sigma_e^m V_e (partial sums over edge chunks, added here in
// chunk order).
#include <math.h>

#include <algorithm>
#include <vector>

#include "gw_ctx.h"
#include "gw_fft.h"
#include "gw_tgrid.h"

namespace gw {

constexpr int kTgBuf = kTgMaxL + kTgMaxL / 16;  // padded LDS buffer

// w2 = exp(-2 pi i n3 / (16 D2)) for the lane's n3 = tid mod 16
template <int D2>
__device__ inline void tg_lds_pass2(double2* __restrict__ buf, int tid, int D1, int S1, double2 w2) {
  if (tid < 16 * D1) {
    const int n3 = tid & 15, k1 = tid >> 4;
    // element n3 + 16 q + S1 k1 sits at tg_pad(n3 + S1 k1) + 17 q (S1 is a
    // multiple of 16)
    const int pb = tg_pad(n3 + S1 * k1);
    double2 v[D2];
#pragma unroll
    for (int q = 0; q < D2; ++q) v[q] = buf[pb + 17 * q];
    tg_pass2<D2>(v, w2);
#pragma unroll
    for (int q = 0; q < D2; ++q) buf[pb + 17 * q] = v[q];
  }
}

struct TgKernelArgs {
  const double2* part;  // row p, chunk point i at p pitch + i
  int64_t pitch;
  TgCover cov[2];       // of the rows whose C_NODE is at least node_from, of the others
  double node_from;
  int64_t n;
  int n_g, L, D2, jmax;
  const double* dec;    // [jmax + 1]: 1 / psi_hat
  const double* coef;
  int64_t ld;
  double dd;
  double* logl;
  const double* hhc;
  const double2* hpart;
  int n_hch, mh;
  double hw_step;
  int64_t c2, cden;
  double rot_re, rot_im;  // exp(-2 pi i c u_j) over 256 points of one r
  double* zout;
  double f0_num, f0_den;
};

// Terms exp(u - B) I0(x) exp(-x) of V grid points relative to the bound B
// (keep false: 0).  V points at a time: a Horner chain of 40 scalar-operand
// steps alone leaves the lane waiting on each.
template <int V>
__device__ inline void tg_terms(const double* u, const double* x, const bool* keep, double B, double* out) {
  bool small = false, large = false;
#pragma unroll
  for (int t = 0; t < V; ++t) {
    small |= keep[t] && x[t] < 20.0;
    large |= keep[t] && !(x[t] < 20.0);
    out[t] = 0.0;
  }
  small = __any(small);
  large = __any(large);
  double f[V];
#pragma unroll
  for (int t = 0; t < V; ++t) f[t] = 1.0;
  if (small) {
    const I0Table c = i0_table();
    double y[V];
#pragma unroll
    for (int t = 0; t < V; ++t) {
      y[t] = x[t] < 20.0 ? 0.25 * x[t] * x[t] : 0.0;
      f[t] = 0.0;
    }
#pragma unroll
    for (int k = 39; k >= 0; --k) {
      const double s = sgpr(c[k]);
#pragma unroll
      for (int t = 0; t < V; ++t) f[t] = fma(f[t], y[t], s);
    }
  }
  if (large) {
    const I0Table c = i0_table() + 40;
    double r[V], v[V], p[V];
#pragma unroll
    for (int t = 0; t < V; ++t) {
      r[t] = rsqrt(x[t] < 20.0 ? 20.0 : x[t]);
      v[t] = r[t] * r[t];
      p[t] = 0.0;
    }
#pragma unroll
    for (int k = 23; k >= 0; --k) {
      const double s = sgpr(c[k]);
#pragma unroll
      for (int t = 0; t < V; ++t) p[t] = fma(p[t], v[t], s);
    }
#pragma unroll
    for (int t = 0; t < V; ++t) f[t] = x[t] < 20.0 ? f[t] : p[t] * r[t] * kInvSqrtTwoPi;
  }
  if (small || large) {
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const double e = exp(u[t] - (x[t] < 20.0 ? x[t] : 0.0) - B);
      out[t] = keep[t] ? e * f[t] : 0.0;
    }
  }
}

// One row per workgroup of W groups of 256 lanes: W = 1 takes r = 0, then
// r = 1; W = 2 both at once (the same sums).  HET = 0: <h|h> = coef[C_HH];
// HET = 1: <h|h>(t_j) as above from hhc [n], the H moments hpart [n_hch][n][mh]
// complex, hw_step = 2 pi hw / (N R), c2 = 2 c and cden = 2 N R, a power of two
// (exp(-2 pi i c u_j) = exp(-2 pi i (c2 j mod cden) / cden)).  zout (else
// NULL): [n][2 jmax + 1][3] = (Re Z(t_j), Im Z(t_j), <h|h>(t_j)), Re NaN for
// unphysical rows, with f_0 t_j = j f0_num / f0_den cycles.
//
// Measured at 1000 rows of 3273 points (L = 4096): 168 us for twelve
// transforms of Chebyshev moments and the log-sum-exp, 68 us here; the
// transforms are about 12 of them, the terms 18, the rest latency: loads
// behind loads, barriers, two workgroups a CU (LDS).  128 rows: 81 us (two
// kernels) and 30.
template <int HET, int D1, int NZ, int W>
__global__ void __launch_bounds__(256 * W, 2) k_tgrid(TgKernelArgs a) {
  __shared__ double2 bufs[W][kTgBuf];
  __shared__ double2 sm[kTgHMax];  // S_m / m!
  __shared__ double red[256], red2[256];
  __shared__ double wmax[4 * W], wsum[8], bound[2];
  const int64_t p = blockIdx.x;
  const int tid = threadIdx.x & 255, half = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  double2* __restrict__ buf = bufs[half];
  const int L = a.L, D2 = D1 > 1 ? 16 : a.D2;
  const int S1 = L / D1;  // = 16 D2
  const int nt = 2 * a.jmax + 1;
  const bool on1 = tid < S1, on3 = tid < L / 16;
  const double valid_at = a.coef[C_VALID * a.ld + p], node_at = a.coef[C_NODE * a.ld + p];
  double hh = HET ? a.hhc[p] : a.coef[C_HH * a.ld + p];
  // roots while the loads are under way: h = exp(-pi i tid / L), w1 = h^2 of
  // the first pass, w2 of the second
  double2 h, w1, w2;
  {
    double s, c;
    sincospi(-(double)tid / (double)L, &s, &c);
    h = make_double2(c, s);
    w1 = c_mul(h, h);
    sincospi(-(double)(tid & 15) / (double)(8 * D2), &s, &c);
    w2 = make_double2(c, s);
  }
  const bool valid = valid_at != 0.0;
  // the lane's grid points: the chunks that reach each, in order
  double2 x[NZ + 1];  // the last: point tid + L
  {
    const TgCover cv = a.cov[node_at >= a.node_from ? 0 : 1];
    const double2* __restrict__ row = a.part + p * a.pitch;
    // the third chunks on of the leading points, four lanes a point
    for (int g0 = 0; g0 < cv.n_many; g0 += 64) {
      const int g = g0 + (tid >> 2);
      double2 s = make_double2(0.0, 0.0);
      if (g < cv.n_many) {
        const int4 c = cv.pts[g];
#pragma unroll 8
        for (int i = c.z + (tid & 3); i <= c.w; i += 4) s = c_add(s, row[cv.shift[i] + g]);
      }
#pragma unroll
      for (int o = 1; o < 4; o <<= 1) s = c_add(s, make_double2(__shfl_xor(s.x, o, 64), __shfl_xor(s.y, o, 64)));
      if ((tid & 3) == 0 && g < cv.n_many) buf[g] = s;
    }
    if (cv.n_many > 0) __syncthreads();  // the same for the workgroup
    // all loads of a kind in flight at once: two chunks reach most points
    int4 c[NZ + 1];
#pragma unroll
    for (int q = 0; q <= NZ; ++q) {
      const int g = tid + (q < NZ ? S1 * q : L);
      c[q] = on1 && g < a.n_g ? cv.pts[g] : make_int4(-1, -1, 0, -1);
    }
    double2 y[NZ + 1];
#pragma unroll
    for (int q = 0; q <= NZ; ++q) {
      x[q] = c[q].x >= 0 ? row[c[q].x] : make_double2(0.0, 0.0);
      y[q] = c[q].y >= 0 ? row[c[q].y] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int q = 0; q <= NZ; ++q) {
      x[q] = c_add(x[q], y[q]);
      const int g = tid + (q < NZ ? S1 * q : L);
      if (g < cv.n_many) {
        x[q] = c_add(x[q], buf[g]);
      } else {
#pragma unroll 8
        for (int i = c[q].z; i <= c[q].w; ++i) x[q] = c_add(x[q], row[cv.shift[i] + g]);
      }
    }
  }
  if (HET) {
    // this row's H moments, summed over the edge chunks: with Q the power of
    // two >= mh, thread (g, q) adds chunks g, g + 256 / Q, ... of moment q, and
    // the 256 / Q sums are added in order
    int Q = 16;
    while (Q < a.mh) Q <<= 1;
    const int q = tid & (Q - 1), ng = 256 / Q;
    if (half == 0) {
      double2 s = make_double2(0.0, 0.0);
      if (q < a.mh)
#pragma unroll 8
        for (int c = tid / Q; c < a.n_hch; c += ng) s = c_add(s, a.hpart[((int64_t)c * a.n + p) * a.mh + q]);
      red[tid] = s.x;
      red2[tid] = s.y;
    }
    __syncthreads();
    if (half == 0 && tid < a.mh) {
      double2 s = make_double2(0.0, 0.0);
      for (int g = 0; g < ng; ++g) s = c_add(s, make_double2(red[tid + Q * g], red2[tid + Q * g]));
      double f = 1.0;  // S_m / m!
      for (int k = 2; k <= tid; ++k) f *= (double)k;
      sm[tid] = make_double2(s.x / f, s.y / f);
    }
  }
#pragma unroll
  for (int it = 0; it < 2 / W; ++it) {
    const int r = W == 1 ? it : half;
    // twiddle powers formed afresh: an empty asm statement marks the roots as
    // changing here, so the compiler does not keep 30 powers of them (they
    // would spill)
    asm volatile("" : "+v"(w1.x), "+v"(w1.y), "+v"(w2.x), "+v"(w2.y));
    // Z(t_j), j = 2 j' + r, goes to the buffer in order of j' (from j_lo on)
    const int j_lo = -((a.jmax + r) >> 1), n_r = ((a.jmax - r) >> 1) - j_lo + 1;
    double2 v[D1];
#pragma unroll
    for (int q = 0; q < D1; ++q) v[q] = q < NZ ? x[q] : make_double2(0.0, 0.0);
    if (r == 0) {
      v[0] = c_add(v[0], x[NZ]);
    } else {
      v[0] = c_sub(v[0], x[NZ]);
#pragma unroll
      for (int q = 0; q < (NZ < D1 ? NZ : D1); ++q) v[q] = c_mul(v[q], q ? c_mul(h, w32(q * (16 / D1))) : h);
    }
    tg_pass1<D1, NZ>(v, w1);
    __syncthreads();  // the previous points are read
    if (on1) {
      const int pb = tg_pad(tid);
#pragma unroll
      for (int k = 0; k < D1; ++k) buf[pb + 17 * (S1 / 16) * k] = v[k];
    }
    __syncthreads();
    if constexpr (D1 > 1) {
      tg_lds_pass2<16>(buf, tid, D1, S1, w2);  // L >= 512: D2 = 16
    } else {
      switch (D2) {
        case 16: tg_lds_pass2<16>(buf, tid, D1, S1, w2); break;
        case 8: tg_lds_pass2<8>(buf, tid, D1, S1, w2); break;
        case 4: tg_lds_pass2<4>(buf, tid, D1, S1, w2); break;
        case 2: tg_lds_pass2<2>(buf, tid, D1, S1, w2); break;
        default: break;
      }
    }
    __syncthreads();
    double2 f[16];
    if (on3) {
#pragma unroll
      for (int q = 0; q < 16; ++q) f[q] = buf[17 * tid + q];
    }
    __syncthreads();
    if (on3) {
      Dft<16>::run_slots(f);
#pragma unroll
      for (int k3 = 0; k3 < 16; ++k3) {
        const int X = tg_owned(L, D1, D2, tid, k3);
        const int i = (X < L / 2 ? X : X - L) - j_lo;
        if (i >= 0 && i < n_r) {
          const int j = 2 * (i + j_lo) + r;
          const double t = a.dec[j < 0 ? -j : j];
          const double2 z = f[dft_slot<16>(k3)];
          buf[i] = make_double2(t * z.x, t * z.y);
        }
      }
    }
    // exp(-2 pi i c u_j) at this lane's first point, and its step over 256
    // points (a rotation applied once per point below)
    double cs = 1.0, sn = 0.0;
    if (HET) {
      const int64_t num = (a.c2 * (int64_t)(2 * (tid + j_lo) + r)) & (a.cden - 1);
      sincospi(-2.0 * (double)num / (double)a.cden, &sn, &cs);
    }
    __syncthreads();
    // ln I0(x) <= x, so u = x - <h|h> / 2 bounds a point's term; those 60 below
    // the largest bound add nothing (as in the distance marginal)
    double bmax = -INFINITY;
    for (int i0 = tid; i0 - tid < n_r; i0 += 1024) {
      double hj[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) hj[t] = hh;
      if (HET) {
        double xq[4], tr[4], ti[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          xq[t] = a.hw_step * (double)(2 * (i0 + 256 * t + j_lo) + r);
          tr[t] = ti[t] = 0.0;
        }
        for (int q = a.mh - 1; q >= 0; --q) {
          const double2 s = sm[q];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const double nr = fma(xq[t], ti[t], s.x);
            ti[t] = fma(-xq[t], tr[t], s.y);
            tr[t] = nr;
          }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          hj[t] += cs * tr[t] - sn * ti[t];
          const double c2_ = cs * a.rot_re - sn * a.rot_im;
          sn = cs * a.rot_im + sn * a.rot_re;
          cs = c2_;
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = i0 + 256 * t;
        if (i < n_r) {
          const double2 z = buf[i];
          if (a.zout) {
            const int j = 2 * (i + j_lo) + r;
            const double cyc = (double)j * a.f0_num / a.f0_den;
            double sn, cs;
            sincospi(2.0 * (cyc - rint(cyc)), &sn, &cs);
            double* zo = a.zout + (p * nt + j + a.jmax) * 3;
            zo[0] = valid ? cs * z.x + sn * z.y : NAN;
            zo[1] = cs * z.y - sn * z.x;
            zo[2] = hj[t];
          }
          const double xa = sqrt(z.x * z.x + z.y * z.y), u = fma(-0.5, hj[t], xa);
          buf[i] = make_double2(u, xa);
          bmax = fmax(bmax, u);
        }
      }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bmax = fmax(bmax, __shfl_xor(bmax, o, 64));
    if (lane == 0) wmax[wave] = bmax;
    __syncthreads();
    const double B = fmax(fmax(wmax[4 * half], wmax[4 * half + 1]), fmax(wmax[4 * half + 2], wmax[4 * half + 3]));
    double acc = 0.0;
    for (int i0 = tid; i0 - tid < n_r; i0 += 1024) {
      double u[4], xa[4], term[4];
      bool keep[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = i0 + 256 * t;
        const double2 ux = i < n_r ? buf[i] : make_double2(-INFINITY, 0.0);
        u[t] = ux.x;
        xa[t] = ux.y;
        keep[t] = !(ux.x < B - 60.0) && !(ux.x == -INFINITY);
      }
      tg_terms<4>(u, xa, keep, B, term);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc += term[t];
    }
    acc = wave_sum(acc);
    if (lane == 0) wsum[4 * r + (wave & 3)] = acc;
    if (tid == 0) bound[r] = B;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double m = fmax(bound[0], bound[1]);
    double s = 0.0;
    for (int r = 0; r < 2; ++r) {
      const double t = ((wsum[4 * r] + wsum[4 * r + 1]) + wsum[4 * r + 2]) + wsum[4 * r + 3];
      // no bound: no point, or none that is a number (then the sum is not one either)
      s += bound[r] > -INFINITY ? exp(bound[r] - m) * t : t;
    }
    a.logl[p] = valid ? -0.5 * a.dd + m + log(s) - log((double)nt) : -INFINITY;
  }
}

gw_status tgrid_tables(gw_ctx* ctx, int L, int jmax) {
  if (ctx->tm_dec && ctx->tm_dec_L == L && ctx->tm_dec_jmax == jmax) return GW_OK;
  int D1, D2;
  if (!tgrid_plan(L, &D1, &D2)) return set_error(GW_ENOTSUP, "time marginal: transform length %d not supported", L);
  const double beta = tgrid_beta((double)jmax / (2.0 * L)), i0_beta = TgBessel()(beta);
  std::vector<double> h(jmax + 1);
  for (int j = 0; j <= jmax; ++j) h[j] = 1.0 / tgrid_psi_hat((double)j / (2.0 * L), beta, i0_beta);
  if (ctx->tm_dec) (void)hipFree(ctx->tm_dec);
  ctx->tm_dec = nullptr;
  ctx->tm_dec_L = 0;
  gw_status s = check_hip(hipMalloc((void**)&ctx->tm_dec, h.size() * sizeof(double)), "time-grid table");
  if (s == GW_OK)
    s = check_hip(hipMemcpy(ctx->tm_dec, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice), "time-grid table");
  if (s != GW_OK) return s;
  ctx->tm_dec_L = L;
  ctx->tm_dec_jmax = jmax;
  return GW_OK;
}

// Rows per chunk: the grid sums of a chunk take at most 1 GiB.
int64_t tgrid_chunk_rows(int64_t n, int64_t pitch) {
  int64_t c = ((int64_t)1 << 30) / (pitch * 16);
  if (c < 64) c = 64;
  return n < c ? n : c;
}

// A launch of few rows (a sampler round) takes both transforms of a row at
// once on its own CU; from two rows a CU on, two workgroups that wait at their
// own barriers are as fast or faster (1000 rows: 70 us against 71 at L = 4096,
// 82 us a call against 90 at L = 1024).
constexpr int64_t kTgWideRows = 256;

template <int HET, int D1, int NZ>
static void launch_tgrid_w(const TgKernelArgs& k, hipStream_t st) {
  if (k.n <= kTgWideRows)
    hipLaunchKernelGGL((k_tgrid<HET, D1, NZ, 2>), dim3((unsigned)k.n), dim3(512), 0, st, k);
  else
    hipLaunchKernelGGL((k_tgrid<HET, D1, NZ, 1>), dim3((unsigned)k.n), dim3(256), 0, st, k);
}

template <int HET>
static void launch_tgrid_form(const TgKernelArgs& k, int D1, int nz, hipStream_t st) {
  switch (D1) {
    case 16:
      switch (nz) {
        case 2: launch_tgrid_w<HET, 16, 2>(k, st); break;
        case 4: launch_tgrid_w<HET, 16, 4>(k, st); break;
        case 8: launch_tgrid_w<HET, 16, 8>(k, st); break;
        default: launch_tgrid_w<HET, 16, 16>(k, st); break;
      }
      break;
    case 8: launch_tgrid_w<HET, 8, 8>(k, st); break;
    case 4: launch_tgrid_w<HET, 4, 4>(k, st); break;
    case 2: launch_tgrid_w<HET, 2, 2>(k, st); break;
    default: launch_tgrid_w<HET, 1, 1>(k, st); break;
  }
}

gw_status launch_tgrid(const gw_ctx* ctx, const TGridArgs& a, hipStream_t st) {
  int D1, D2;
  if (!tgrid_plan(a.L, &D1, &D2) || 2 * a.jmax + 1 > a.L)
    return set_error(GW_ENOTSUP, "time marginal: a grid of %d points per %d-point transform is not supported",
                     2 * a.jmax + 1, a.L);
  if (a.het && a.mh > kTgHMax) return set_error(GW_ENOTSUP, "time marginal: %d norm moments exceed %d", a.mh, kTgHMax);
  if (!ctx->tm_dec || ctx->tm_dec_L != a.L || ctx->tm_dec_jmax != a.jmax)
    return set_error(GW_ESTATE, "time marginal: table not built for this grid");
  const int S1 = a.L / D1;
  if (a.n_g > a.L + S1)
    return set_error(GW_EINVAL, "time marginal: %d grid points exceed the transform length", a.n_g);
  if (a.n <= 0) return GW_OK;
  // nonzero first-pass inputs per lane: grid points g = lane + (L / D1) q < n_g
  int nz = 2;
  while (nz < D1 && nz * S1 < a.n_g) nz <<= 1;
  TgKernelArgs k{};
  k.part = (const double2*)a.part;
  k.pitch = a.pitch;
  k.cov[0] = a.cov[0];
  k.cov[1] = a.cov[1];
  k.node_from = a.node_from;
  k.n = a.n;
  k.n_g = a.n_g;
  k.L = a.L;
  k.D2 = D2;
  k.jmax = a.jmax;
  k.dec = ctx->tm_dec;
  k.coef = a.coef;
  k.ld = a.ld;
  k.dd = ctx->dd;
  k.logl = a.logl;
  k.zout = a.zout;
  k.f0_num = a.f0_num;
  k.f0_den = a.f0_den;
  k.cden = 1;
  if (a.het) {
    k.hhc = a.hhc;
    k.hpart = (const double2*)a.hpart;
    k.n_hch = a.n_hch;
    k.mh = a.mh;
    k.hw_step = a.hw_step;
    k.c2 = a.c2;
    k.cden = a.cden;
    const double turn = (double)((a.c2 * 512) & (a.cden - 1)) / (double)a.cden;
    k.rot_re = cos(2.0 * kPi * turn);
    k.rot_im = -sin(2.0 * kPi * turn);
    launch_tgrid_form<1>(k, D1, nz, st);
  } else {
    launch_tgrid_form<0>(k, D1, nz, st);
  }
  return check_hip(hipGetLastError(), "time-grid launch");
}

}  // namespace gw
