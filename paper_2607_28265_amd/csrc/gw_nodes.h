// Interpolation nodes of the full-band sums.
//
// Every full-band sum is linear in samples of a smooth function of frequency,
//   z_i = sum_k u_ik G_i(f_k),   G_i(f) = exp(-2 pi i (Psi(f) + f tau_i)),
// with weights u_ik that depend on the data alone.  Relative to a fixed
// reference phase R(f), G_i turns by at most S(f) = |Psi' + tau_i - R'| cycles
// per Hz, and on a long segment that is far below one turn per bin over most
// of the band (a 128 s segment samples every 1/128 Hz what a signal of under
// two seconds does above 100 Hz).  On a block of bins on which
// G_i exp(2 pi i R) turns by omega radians to either side of the centre, its
// polynomial interpolant at n Chebyshev nodes errs by less than about
// 2 (omega / 2)^n / n!, so with
//   W_ij = sum_k l_j(f_k) u_ik exp(-2 pi i R(f_k))
// (l_j the Lagrange polynomials of the block's nodes)
//   z_i = sum_j W_ij G_i(f_j) exp(2 pi i R(f_j))
// to 1e-13 of the block's sum of |u_ik|: the same sums from n samples a block
// instead of one per bin.  The weights are computed once per context.  A block
// on which that saves less than a tenth keeps its bins (a node per bin).
//
// R is half the phase of a reference waveform of chirp mass kNodeMc: chirp
// times run from 0 (heavy binaries) to that waveform's, so half of it halves
// the largest S.  S is the largest of a set of waveforms around the sampler's
// prior (kNodeMc and 1.45 Msun, the prior's mass ratios and tides, aligned
// spins of 0.1), times 1.02, plus 1 ms.  k_prologue compares each row's
// Psi' - R' with S at kNodeCheck frequencies and its delays with tau_max; a row
// that exceeds either takes the sums over every bin instead.  Between those
// frequencies Psi' - R' may exceed S (a search over masses, spins and tides found
// up to 9 % on 20-2048 Hz, 12 % on 1-8192 Hz), but S + tau_max by under 2 %, and
// the node counts have more to spare: their bound is far above the error at tens
// of nodes, and they take one node more.  Such rows interpolate to 7e-14 like the
// rest.
#pragma once

#include "gw_device.h"
#include "gw_trig_fit.h"

namespace gw {

constexpr double kNodeMc = 1.05;   // Msun
constexpr double kNodeTol = 1e-13; // interpolation error per unit sum of |u|
constexpr int kNodeMax = 128;      // most nodes of a block
constexpr int kNodeCheck = 24;     // frequencies of the row check

constexpr double kTauCap = 0.25;   // s, delays of the wide table and of the waveform cache

// Values of the coefficient column C_NODE: the row's phase lies within what
// the tables are built for, and its delays within neither table's, the wide
// table's (kTauCap) or the context's own (tau_max).  Zero: the phase does not.
constexpr double kNodePhase = 1.0, kNodeWide = 2.0, kNodeFull = 3.0;
// A waveform cache's row whose slot holds no waveform.
constexpr double kNodeNoSlot = -1.0;

// The row check's frequencies: x = f^(1/3), ln f, x^-8, x^-3, R'(f), S(f).
struct NodeCheck {
  double v[kNodeCheck][6];
  double tau_max;  // s
};

// The tables of a reduction and the C_NODE value of the rows each covers.
struct NodeTabs {
  const double* rec[2];
  int n[2];
  double row[2];
};

// Record of one node: x, x^2, f^(-5/3), ln f, f, R (cycles), then Re, Im W_i
// per detector.
__host__ __device__ constexpr int node_rs(int nd) { return 6 + 2 * nd; }

// Rows to a tile of 64 lanes, covered rows apart from the others: a wave that
// holds both kinds pays for both, and two rows in a hundred beyond the tables put
// one into most tiles (20,000 such rows of 8 s, plain mixed: 216 us a call, 149 so;
// 99 with none of them beyond, 144 with all).  In a group of kTileGroup tiles the covered rows come first, each kind in
// order, so one tile at most is mixed.  k_prologue leaves each tile's mask of
// covered rows in C_TILE of its first row; a group of one kind is taken as it lies.
constexpr int kTileGroup = 16;

struct TileRow {
  int64_t p;     // n: no row
  bool covered;
};

// The row of lane ``lane`` of tile ``tile`` (of the n rows at coef, stride ld).  All
// lanes of the wave together.
__device__ inline TileRow tile_row(const double* __restrict__ coef, int64_t ld, int64_t n, int64_t tile, int lane) {
  const int64_t base = tile / kTileGroup * kTileGroup * 64;
  const int rows = n - base < kTileGroup * 64 ? (int)(n - base) : kTileGroup * 64;
  int k = (int)(tile % kTileGroup) * 64 + lane;
  const bool none = k >= rows;  // (no lane leaves: the words below come from all)
  // lane i: the masks of tile i of the group
  uint64_t in = 0, out = 0;
  if (lane * 64 < rows) {
    in = (uint64_t)__double_as_longlong(coef[C_TILE * ld + base + 64 * lane]);
    const int left = rows - 64 * lane;
    out = ~in & (left >= 64 ? ~0ull : (1ull << left) - 1);
  }
  const bool any_in = __any(in != 0), any_out = __any(out != 0);
  if (!any_in || !any_out) return TileRow{none ? n : base + k, !none && any_in};
  int covered = __popcll(in);
#pragma unroll
  for (int o = 1; o < kTileGroup; o <<= 1) covered += __shfl_xor(covered, o, 64);
  covered = __builtin_amdgcn_readfirstlane(covered);
  const bool kind = k < covered;
  if (!kind) k -= covered;
  // the k-th row of its kind: its tile, then its bit
  uint64_t word = 0;
  int at = -1;
#pragma unroll
  for (int i = 0; i < kTileGroup; ++i) {
    const uint32_t il = __builtin_amdgcn_readlane((uint32_t)in, i), ih = __builtin_amdgcn_readlane((uint32_t)(in >> 32), i);
    const uint32_t ol = __builtin_amdgcn_readlane((uint32_t)out, i), oh = __builtin_amdgcn_readlane((uint32_t)(out >> 32), i);
    const uint64_t w = kind ? (uint64_t)ih << 32 | il : (uint64_t)oh << 32 | ol;
    const int c = __popcll(w);
    if (at < 0 && k < c) {
      at = i;
      word = w;
    } else if (at < 0) {
      k -= c;
    }
  }
  int bit = 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int c = __popcll(word & ((1ull << o) - 1));
    if (k >= c) {
      k -= c;
      word >>= o;
      bit += o;
    }
  }
  return TileRow{none ? n : base + 64 * at + bit, !none && kind};
}

// d Psi / d f without the linear time term, in cycles per Hz.
__device__ inline double phase_slope(const PhaseCoef& c, double x, double lnf, double xm8, double xm3) {
  // sum_j a_j (j - 5) / 3 x^(j - 8) + (b5 + b6 x) / f + b6 ln f / (3 x^2)
  double t = fma(x * x, c.a12 * (7.0 / 3.0), c.a10 * (5.0 / 3.0));
  t = x * x * t;
  t = fma(x, t, c.a7 * (2.0 / 3.0));
  t = fma(x, t, c.a6 * (1.0 / 3.0));
  t = x * t;
  t = fma(x, t, c.a4 * (-1.0 / 3.0));
  t = fma(x, t, c.a3 * (-2.0 / 3.0));
  t = fma(x, t, -c.a2);
  t = fma(x * x, t, c.a0 * (-5.0 / 3.0));
  const double l = fma(c.b6 * x, fma(lnf, 1.0 / 3.0, 1.0), c.b5);
  return fma(l, xm3, t * xm8);
}

// exp(-2 pi i r) at a node.  FP64 form: the full-accuracy pair.  Mixed form:
// FP64 polynomials good to 2e-11 / 1.2e-10, where the walk over bins takes the
// FP32 hardware pair (6e-8): with tens of bins behind each node the rounding
// of the phasors averages over that many fewer samples, and the difference
// costs 5 of the 84 instructions of a node.
template <int PREC>
__device__ inline void node_phasor(double r, const TrigConsts& T, const TrigFit& F, double* gr, double* gi) {
  if (PREC == 0) {
    double s, c;
    sincos_cycles(r, T, &s, &c);
    *gr = c;
    *gi = -s;
  } else {
    const double t = r - rint(r);
    const double s = t * t;
    double a = F.s[7], b = F.c[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) {
      a = fma(a, s, F.s[k]);
      b = fma(b, s, F.c[k]);
    }
    *gr = b;
    *gi = -(t * a);
  }
}

// Phase at a node relative to the reference, cycles.
__device__ inline double node_phase(const PhaseCoef& c, double x, double x2, double xm5, double lnf, double ref) {
  double t = fma(x2, c.a12, c.a10);
  t = fma(x2, t, c.a8);
  t = fma(x, t, c.a7);
  t = fma(x, t, c.a6);
  t = fma(x, t, c.a5);
  t = fma(x, t, c.a4);
  t = fma(x, t, c.a3);
  t = fma(x, t, c.a2);
  t = fma(x2, t, c.a0);
  const double lg = fma(c.b6, x, c.b5);
  return fma(lg, lnf, fma(t, xm5, -ref));
}

}  // namespace gw
