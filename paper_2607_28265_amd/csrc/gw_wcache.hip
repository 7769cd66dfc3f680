// Waveform cache as a library object: the paper's pair of a slow likelihood
// (regenerates and caches the waveform) and a fast one (reuses it, Sec. III.B
// and Sec. III.A: the fast blocks only redo the detector projection and the
// marginalisations).  The sampler's sweep keeps the same cache internally;
// this entry point lets any caller use it.
#include <string.h>

#include "gw_ctx.h"

using namespace gw;

struct gw_wcache {
  gw_ctx* ctx = nullptr;
  int64_t n_slots = 0;
  int64_t slot_f2 = 0;
  float2* wc = nullptr;  // [n_slots][slot_f2] block moments (FP32 complex)
  double* zc = nullptr;  // [n_slots][2 n_det] sums z_i of each slot's point
  double* rec = nullptr;  // [n_slots][kSlotRec] each slot's phase coefficients and what it holds
  int32_t* owner = nullptr;  // [n_slots]: -1 between calls
  // per-call workspace: zrow [cap][2 kMaxDet], sl [cap] (checked slots), and
  // the slots whose moments are wanted with their rows, bslot and brow [cap],
  // bcount of them
  int64_t cap = 0;
  char* mem = nullptr;
  double* zrow = nullptr;
  int32_t* sl = nullptr;
  int32_t* bslot = nullptr;
  int32_t* brow = nullptr;
  int32_t* bcount = nullptr;
};

namespace {

__global__ void k_wc_fill(int32_t* __restrict__ a, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// sl[r] = slots[r] when 0 <= slots[r] < n_slots, else -1; the largest row
// naming each slot claims it.  Clears the list of moments to build.
__global__ void k_wc_slots(const int32_t* __restrict__ slots, int64_t n, int64_t n_slots, int32_t* __restrict__ sl,
                           int32_t* __restrict__ owner, int32_t* __restrict__ bcount) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r == 0) *bcount = 0;
  if (r >= n) return;
  const int32_t s = slots[r];
  const bool ok = s >= 0 && s < n_slots;
  sl[r] = ok ? s : -1;
  if (ok) atomicMax(&owner[s], (int32_t)r);
}

// The claiming row of each slot stores its sums, zc[sl[r]] = zrow[r], and its
// phase coefficients, and asks for the slot's moments when no node table covers
// its phase: the fast rows of the other slots are summed over the nodes.  What
// the slot holds is stored with it, so that the fast rows ask for nothing else.
// (The list's order does not matter: each slot's moments come from its own row.)
__global__ void k_wc_store(const double* __restrict__ zrow, const int32_t* __restrict__ sl,
                           const int32_t* __restrict__ owner, const double* __restrict__ coef, int64_t n, int nd,
                           bool nodes, double* __restrict__ zc, double* __restrict__ rec,
                           int32_t* __restrict__ bslot,
                           int32_t* __restrict__ brow, int32_t* __restrict__ bcount) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int32_t s = sl[r];
  if (s < 0 || owner[s] != (int32_t)r) return;
  for (int j = 0; j < 2 * nd; ++j) zc[(int64_t)s * 2 * nd + j] = zrow[r * 2 * nd + j];
  double* __restrict__ w = rec + (int64_t)s * kSlotRec;
#pragma unroll
  for (int j = 0; j < kSlotRec - 1; ++j) w[j] = coef[kSlotCols[j] * n + r];
  // a row that is not physical has zero coefficients, which moments serve
  const bool covered = nodes && coef[C_VALID * n + r] != 0.0 && coef[C_NODE * n + r] >= kNodePhase;
  w[kSlotRec - 1] = covered ? kSlotNodes : kSlotMoments;
  if (covered) return;
  const int32_t q = atomicAdd(bcount, 1);
  bslot[q] = s;
  brow[q] = (int32_t)r;
}

// Release the claims (owner back to -1) once the slots are written; rows whose
// slot is out of range get log L = NaN.
__global__ void k_wc_release(const int32_t* __restrict__ sl, int64_t n, int32_t* __restrict__ owner,
                             double* __restrict__ logl) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  if (sl[r] >= 0) owner[sl[r]] = -1;
  else logl[r] = __builtin_nan("");
}

// sl[r] = slots[r], or -1 when that is no slot.
__global__ void k_wc_clip(const int32_t* __restrict__ slots, int64_t n, int64_t n_slots, int32_t* __restrict__ sl) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n) sl[r] = slots[r] >= 0 && slots[r] < n_slots ? slots[r] : -1;
}

// Rows whose slot is out of range or was never written get log L = NaN.
__global__ void k_wc_mark(const double* __restrict__ coef, int64_t n, double* __restrict__ logl) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n && coef[C_NODE * n + r] == kNodeNoSlot) logl[r] = __builtin_nan("");
}

gw_status wc_reserve(gw_wcache* c, int64_t n) {
  gw_status s = cached_reserve(c->ctx, n);
  if (s != GW_OK || c->cap >= n) return s;
  if (c->mem) (void)hipFree(c->mem);
  c->mem = nullptr;
  c->cap = 0;
  const size_t bytes = (size_t)n * 2 * kMaxDet * sizeof(double) + 3 * (size_t)n * sizeof(int32_t) + sizeof(int32_t);
  s = check_hip(hipMalloc((void**)&c->mem, bytes), "waveform cache workspace");
  if (s != GW_OK) return s;
  c->zrow = (double*)c->mem;
  c->sl = (int32_t*)(c->mem + (size_t)n * 2 * kMaxDet * sizeof(double));
  c->bslot = c->sl + n;
  c->brow = c->bslot + n;
  c->bcount = c->brow + n;
  c->cap = n;
  return GW_OK;
}

gw_status wc_check(const gw_wcache* c, const double* theta, const int32_t* slots, int64_t n, int32_t marg,
                   int32_t prec, const double* logl, const char* who) {
  if (!c) return set_error(GW_EINVAL, "%s: cache is NULL", who);
  if (n < 0) return set_error(GW_EINVAL, "%s: n < 0", who);
  if (n > 0 && (!theta || !slots || !logl)) return set_error(GW_EINVAL, "%s: null pointer", who);
  if (n > 0x7fffffff) return set_error(GW_EINVAL, "%s: n too large", who);
  if (marg < GW_MARG_NONE || marg > GW_MARG_PHASE_DIST) return set_error(GW_EINVAL, "%s: bad marg=%d", who, marg);
  if (prec != GW_PREC_FP64 && prec != GW_PREC_MIXED) return set_error(GW_EINVAL, "%s: bad prec=%d", who, prec);
  if (marg == GW_MARG_PHASE_DIST && c->ctx->n_dist <= 0)
    return set_error(GW_ESTATE, "%s: distance marginal needs a distance grid", who);
  return GW_OK;
}

}  // namespace

extern "C" {

gw_status gw_wcache_create(gw_ctx* ctx, int64_t n_slots, gw_wcache** out) {
  if (!out) return set_error(GW_EINVAL, "gw_wcache_create: out is NULL");
  *out = nullptr;
  if (!ctx) return set_error(GW_EINVAL, "gw_wcache_create: ctx is NULL");
  if (n_slots < 1) return set_error(GW_EINVAL, "gw_wcache_create: n_slots < 1");
  const int64_t f2 = wmom_slot_f2(ctx);
  if ((double)n_slots * (double)f2 * sizeof(float2) > 128.0 * (1ull << 30))
    return set_error(GW_EINVAL, "gw_wcache_create: %lld slots of %lld bytes exceed 128 GiB", (long long)n_slots,
                     (long long)(f2 * sizeof(float2)));
  gw_status s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s == GW_OK) s = nodes_wide_init(ctx);
  if (s != GW_OK) return s;
  gw_wcache* c = new (std::nothrow) gw_wcache();
  if (!c) return set_error(GW_ENOMEM, "gw_wcache_create");
  c->ctx = ctx;
  c->n_slots = n_slots;
  c->slot_f2 = f2;
  s = check_hip(hipMalloc((void**)&c->wc, (size_t)n_slots * f2 * sizeof(float2)), "waveform cache");
  if (s == GW_OK)
    s = check_hip(hipMalloc((void**)&c->zc, (size_t)n_slots * 2 * ctx->n_det * sizeof(double)), "cached sums");
  if (s == GW_OK)
    s = check_hip(hipMalloc((void**)&c->rec, (size_t)n_slots * kSlotRec * sizeof(double)), "slot records");
  if (s == GW_OK) s = check_hip(hipMemset(c->rec, 0, (size_t)n_slots * kSlotRec * sizeof(double)), "slot records");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&c->owner, (size_t)n_slots * sizeof(int32_t)), "slot claims");
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_wc_fill, dim3((unsigned)((n_slots + 255) / 256)), dim3(256), 0, nullptr, c->owner, n_slots,
                       -1);
    s = check_hip(hipGetLastError(), "slot claims fill");
  }
  if (s == GW_OK) s = check_hip(hipDeviceSynchronize(), "waveform cache set-up");
  if (s != GW_OK) {
    if (c->wc) (void)hipFree(c->wc);
    if (c->zc) (void)hipFree(c->zc);
    if (c->rec) (void)hipFree(c->rec);
    if (c->owner) (void)hipFree(c->owner);
    delete c;
    return s;
  }
  *out = c;
  return GW_OK;
}

gw_status gw_wcache_destroy(gw_wcache* c) {
  if (!c) return GW_OK;
  (void)hipSetDevice(c->ctx->device);
  if (c->wc) (void)hipFree(c->wc);
  if (c->zc) (void)hipFree(c->zc);
  if (c->rec) (void)hipFree(c->rec);
  if (c->owner) (void)hipFree(c->owner);
  if (c->mem) (void)hipFree(c->mem);
  delete c;
  return GW_OK;
}

gw_status gw_wcache_update(gw_wcache* c, const double* theta, const int32_t* slots, int64_t n, int32_t marg,
                           int32_t prec, double* logl, void* stream) {
  gw_status s = wc_check(c, theta, slots, n, marg, prec, logl, "gw_wcache_update");
  if (s != GW_OK || n == 0) return s;
  gw_ctx* ctx = c->ctx;
  hipStream_t st = (hipStream_t)stream;
  s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s == GW_OK) s = wc_reserve(c, n);
  if (s != GW_OK) return s;
  int tpb, nch;
  cached_shape(ctx, &tpb, &nch);
  const unsigned blocks = (unsigned)((n + 255) / 256);
  s = launch_prologue(ctx, theta, n, marg, ctx->coef, n, st);
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_wc_slots, dim3(blocks), dim3(256), 0, st, slots, n, c->n_slots, c->sl, c->owner, c->bcount);
    s = check_hip(hipGetLastError(), "slot check launch");
  }
  const int nn = cached_node_chunks(ctx, n, nch);
  if (s == GW_OK) s = launch_all_rows(ctx, ctx->coef, n, prec, nch, nn, ctx->partial, st);
  if (s == GW_OK)
    s = launch_epilogue_cached(ctx, ctx->partial, nch, nn, ctx->coef, n, n, marg, prec,
                               logl, nullptr, nullptr, c->zrow, st);
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_wc_store, dim3(blocks), dim3(256), 0, st, c->zrow, c->sl, c->owner, ctx->coef, n, ctx->n_det,
                       ctx->nodes.n > 0, c->zc, c->rec, c->bslot, c->brow, c->bcount);
    s = check_hip(hipGetLastError(), "cached sums launch");
  }
  if (s == GW_OK) s = launch_wmom_build(ctx, ctx->coef, n, c->bslot, c->bcount, n, 1, c->brow, prec, c->wc, st);
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_wc_release, dim3(blocks), dim3(256), 0, st, c->sl, n, c->owner, logl);
    s = check_hip(hipGetLastError(), "slot release launch");
  }
  return s;
}

gw_status gw_wcache_loglike(gw_wcache* c, const double* theta, const int32_t* slots, int64_t n, int32_t kind,
                            int32_t marg, int32_t prec, double* logl, void* stream) {
  gw_status s = wc_check(c, theta, slots, n, marg, prec, logl, "gw_wcache_loglike");
  if (s != GW_OK || n == 0) return s;
  if (kind != 1 && kind != 2) return set_error(GW_EINVAL, "gw_wcache_loglike: kind must be 1 or 2");
  gw_ctx* ctx = c->ctx;
  hipStream_t st = (hipStream_t)stream;
  s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s == GW_OK) s = wc_reserve(c, n);
  if (s != GW_OK) return s;
  int tpb, nch;
  cached_shape(ctx, &tpb, &nch);
  const unsigned blocks = (unsigned)((n + 255) / 256);
  s = launch_prologue_slots(ctx, theta, n, marg, slots, SlotWaves{c->rec, c->n_slots}, ctx->coef, n, st);
  if (s != GW_OK) return s;
  // out-of-range slots read slot 0 and are marked NaN afterwards
  if (kind == 2) {  // the slots' sums, no reduction
    hipLaunchKernelGGL(k_wc_clip, dim3(blocks), dim3(256), 0, st, slots, n, c->n_slots, c->sl);
    s = check_hip(hipGetLastError(), "slot check launch");
    if (s == GW_OK)
      s = launch_epilogue_cached(ctx, ctx->partial, 0, 0, ctx->coef, n, n, marg, prec, logl, c->sl, c->zc, nullptr, st);
  } else {
    const int cm = wcache_fast_chunks(ctx, nch), nn = cached_node_chunks(ctx, n, nch, true);
    s = launch_wcache_fast(ctx, ctx->coef, n, prec, cm, nn, slots, c->n_slots, c->wc, ctx->partial, st);
    if (s == GW_OK)
      s = launch_epilogue_z(ctx, ctx->partial, cm, nn, ctx->coef, n, n, marg, prec, logl, nullptr, nullptr, nullptr,
                            ctx->zbuf, st, kNodeWide);
  }
  if (s == GW_OK) {
    hipLaunchKernelGGL(k_wc_mark, dim3(blocks), dim3(256), 0, st, ctx->coef, n, logl);
    s = check_hip(hipGetLastError(), "slot check launch");
  }
  return s;
}

}  // extern "C"
