// Launch-shape tuner for the pair kernels.
//
// Candidates (targets per lane, symmetric or ordered evaluation, source split / work-item size,
// workgroup count) are timed with HIP events on the caller's configuration and the fastest is
// kept in the context; single-system and batched products have fields of their own.  Results
// are cached per (precision, single or batched, log2 of the sphere count and, for single float64
// systems, whether the tile follows tpt and whether there is a box), so a later call with a similar problem reuses the choice
// without timing.
#include <algorithm>
#include <cmath>
#include <vector>

#include "rpb_internal.h"

namespace rpb {

namespace {

using Key = std::tuple<int, int, int, int>;   // precision, batched, log2(n), float64 tile rule

std::map<Key, Tuning> &cache(rpb_ctx *ctx) { return ctx->tune_cache; }

int time_candidate(rpb_ctx *ctx, const rpb_params *p, int32_t nsys, const int64_t *offs,
                   const double *pos, int reps, bool expanded, hipStream_t stream,
                   double *ms_out) {
  const int64_t n = offs[nsys];
  int st;
  double *vel =
      static_cast<double *>(workspace(ctx, WS_VEC_A, size_t(3 * n) * sizeof(double), &st));
  if (!vel) return st;
  Packed g;
  RPB_TRY(pack_geometry(ctx, p, n, pos, WS_GEOM, &g, stream));
  Batch b;
  if (nsys > 1) RPB_TRY(prepare_batch(ctx, nsys, offs, p->precision, &b, stream));
  // the positions serve as a finite source vector: only the time matters here
  auto once = [&]() -> int {
    return nsys > 1 ? matvec_batched(ctx, p, b, g, pos, nullptr, nullptr, vel, stream)
                    : matvec_packed(ctx, p, g, pos, nullptr, 0, n, vel, stream, nullptr, expanded);
  };
  RPB_TRY(once());
  hipEvent_t e0, e1;
  RPB_HIP(ctx, hipEventCreate(&e0));
  RPB_HIP(ctx, hipEventCreate(&e1));
  int rc = hipEventRecord(e0, stream) == hipSuccess ? RPB_OK : RPB_EDEVICE;
  for (int r = 0; r < reps && rc == RPB_OK; ++r) rc = once();
  float ms = 0.0f;
  if (rc == RPB_OK && (hipEventRecord(e1, stream) != hipSuccess ||
                       hipEventSynchronize(e1) != hipSuccess ||
                       hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
    rc = fail(ctx, RPB_EDEVICE, "tuning timer failed");
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *ms_out = ms / reps;
  return rc;
}

// The fastest of `cands` for precision q.  Those within a quarter of the fastest are timed twice more,
// in turn, and the fastest time of each counts: candidates differ by a few per cent, and a time
// taken once can be off by more (a clock change in between made a 65,536-sphere benchmark run with
// four targets per lane at 59.3 ms a step, 55.9 with the two that other runs chose).
int rank_candidates(rpb_ctx *ctx, const rpb_params *p, int32_t nsys, const int64_t *offs,
                    const double *pos, int reps, int q, bool expanded,
                    const std::vector<Shape> &cands, hipStream_t stream, Shape *best,
                    double *best_ms) {
  std::vector<double> ms(cands.size(), -1.0);
  for (int round = 0; round < 3; ++round) {
    const double limit = round > 0 ? 1.25 * *std::min_element(ms.begin(), ms.end()) : 0.0;
    for (size_t i = 0; i < cands.size(); ++i) {
      if (round > 0 && ms[i] > limit) continue;
      ctx->tune.s[q] = cands[i];
      double t = 0.0;
      RPB_TRY(time_candidate(ctx, p, nsys, offs, pos, reps, expanded, stream, &t));
      ms[i] = round > 0 ? std::min(ms[i], t) : t;
    }
  }
  const size_t i = size_t(std::min_element(ms.begin(), ms.end()) - ms.begin());
  *best = cands[i];
  *best_ms = ms[i];
  return RPB_OK;
}

}  // namespace

}  // namespace rpb

using namespace rpb;

extern "C" {

int rpb_get_tuning(const rpb_ctx *ctx, rpb_tuning *out) {
  if (!ctx || !out) return RPB_EINVAL;
  rpb_shape *dst[2] = {&out->fp64, &out->mixed};
  for (int q = 0; q < 2; ++q) {
    const Shape &v = ctx->tune.s[q];
    *dst[q] = rpb_shape{v.tpt,       v.target_wgs, v.batch_chunk,    v.batch_wgs,
                        v.symmetric, v.batch_tpt,  v.batch_symmetric};
  }
  return RPB_OK;
}

int rpb_set_tuning(rpb_ctx *ctx, const rpb_tuning *t) {
  if (!ctx || !t) return RPB_EINVAL;
  const rpb_shape *src[2] = {&t->fp64, &t->mixed};
  for (int q = 0; q < 2; ++q) {
    const rpb_shape &v = *src[q];
    if ((v.tpt != 1 && v.tpt != 2 && v.tpt != 4) || v.target_wgs < 1 || v.target_wgs > (1 << 20) ||
        v.batch_chunk < 256 || v.batch_chunk % 256 != 0 || v.batch_chunk > (1 << 20) ||
        v.batch_wgs < 1 || v.batch_wgs > (1 << 20) || (v.symmetric != 0 && v.symmetric != 1) ||
        (v.batch_tpt != 1 && v.batch_tpt != 2) ||
        (v.batch_symmetric != 0 && v.batch_symmetric != 1))
      return fail(ctx, RPB_EINVAL, "tuning values out of range");
  }
  for (int q = 0; q < 2; ++q) {
    const rpb_shape &v = *src[q];
    Shape &s = ctx->tune.s[q];
    s = Shape{v.tpt,       v.target_wgs, v.batch_chunk,     v.batch_wgs,
              v.symmetric, v.batch_tpt,  v.batch_symmetric, s.tpt == v.tpt ? s.drift_tpt : v.tpt};
  }
  return RPB_OK;
}

int rpb_autotune(rpb_ctx *ctx, const rpb_params *p, int32_t nsys, const int64_t *offs,
                 const double *pos, int reps, rpb_tuning *out, double *best_ms_out,
                 rpb_stream_t stream_) {
  RPB_TRY(check_params(ctx, p));
  RPB_TRY(check_offsets(ctx, nsys, offs));
  if (nsys > 1 && p->lx > 0.0)
    return fail(ctx, RPB_EINVAL, "pseudo-periodic boundaries are supported for single systems");
  if (reps < 1 || reps > 100) return fail(ctx, RPB_EINVAL, "reps must be in [1, 100]");
  const int64_t n = offs[nsys];
  if (n == 0) return fail(ctx, RPB_EINVAL, "nothing to tune");
  if (!pos) return fail(ctx, RPB_EINVAL, "pos must not be NULL");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  RPB_HIP(ctx, hipSetDevice(ctx->device));
  RPB_TRY(check_finite(ctx, pos, n, stream));
  const bool batched = nsys > 1;
  const int q = p->precision == RPB_FP64 ? RPB_FP64 : RPB_MIXED;
  // Float64 products of single systems.  Where the tile follows tpt, one target per lane loses without
  // a box (8,191 spheres: 135 us against 118, 16,384: 453 against 376; free space: 96 against 82,
  // 298 against 230) and is not offered; in a box it wins at some sizes (8,191: 722 against 793,
  // 12,000: 1,740 against 1,587), so it is.  Below that size both are the same launch, and two stands.
  // The drift of mixed steps has its own count (4,099 spheres: 127 us with one, 148 with two; 8,191:
  // 286 and 300; 16,384: 960 and 902).
  const bool f64 = q == RPB_FP64 && !batched, box = p->lx > 0.0;
  const bool follows = f64 && f64_tile_follows_tpt(n);
  const Key key{q, batched ? 1 : 0, int(std::floor(std::log2(double(n)))),
                f64 ? (follows ? 1 : 0) + (box ? 2 : 0) : 0};
  auto &tab = cache(ctx);
  double best_ms = -1.0;
  auto it = tab.find(key);
  if (it != tab.end()) {
    ctx->tune.s[q] = it->second.s[q];
  } else {
    const Shape base = ctx->tune.s[q];
    const bool timing = ctx->timing;
    ctx->timing = false;
    Shape best = base;
    std::vector<Shape> cands;
    for (int tpt : {1, 2}) {
      // a system within one tile of 256 targets (one per lane of a 256-lane workgroup): two
      // targets per lane would leave half of each lane's targets empty
      if (!batched && tpt == 2 && n <= 256) continue;
      if (batched) {
        for (int wgs : {1024, 2048, 4096}) {
          Shape c = base;
          c.batch_tpt = tpt;
          c.batch_wgs = wgs;
          c.batch_symmetric = 1;
          cands.push_back(c);
          c.batch_symmetric = 0;
          for (int chunk : {512, 1024, 2048}) {
            c.batch_chunk = chunk;
            cands.push_back(c);
          }
        }
      } else {
        Shape c = base;
        c.tpt = tpt;
        c.symmetric = 1;
        if (!f64 || tpt == 2 || n <= 256 || (follows && box)) cands.push_back(c);
        c.symmetric = 0;
        for (int wgs : {2048, 4096, 8192, 16384}) {
          c.target_wgs = wgs;
          cands.push_back(c);
        }
      }
    }
    if (!batched && q == RPB_MIXED && n >= 4 * 1024) {   // 4 targets per lane: tiles of 1,024
      // spheres, mixed symmetric kernel only (float64 products choose their tile by size, and the
      // drift of mixed steps is 15 % slower with it); on smaller systems most lanes would idle
      Shape c = base;
      c.tpt = 4;
      c.symmetric = 1;
      cands.push_back(c);
    }
    int rc = rank_candidates(ctx, p, nsys, offs, pos, reps, q, false, cands, stream, &best, &best_ms);
    if (rc == RPB_OK && f64) {
      cands.clear();
      for (int tpt : {1, 2}) {
        if (tpt == 2 && n <= 256) continue;
        Shape c = base;
        c.symmetric = 1;
        c.drift_tpt = tpt;
        cands.push_back(c);
      }
      Shape drift = base;
      double ms = 0.0;
      rc = rank_candidates(ctx, p, nsys, offs, pos, reps, q, true, cands, stream, &drift, &ms);
      best.drift_tpt = drift.drift_tpt;
    }
    ctx->timing = timing;
    ctx->tune.s[q] = rc == RPB_OK ? best : base;
    if (rc != RPB_OK) return rc;
    tab[key] = ctx->tune;
  }
  if (best_ms_out) *best_ms_out = best_ms;
  return rpb_get_tuning(ctx, out);
}

}  // extern "C"
