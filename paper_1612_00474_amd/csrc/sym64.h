// Float64 symmetric tile pairs, one or several source vectors: U_v = M F_v (+ M_C T for v = 0)
// with one evaluation per unordered pair of spheres.
//
// A workgroup of W wavefronts owns the tile pair (I, J), I <= J, of tiles of TS = 64 WT TPT
// spheres.  The wavefronts stand WT along the targets of tile I (TPT targets per lane) and
// WS = W / WT along the rotation: sources are taken in blocks of 64, at rotation step k lane l
// works on source (l + k) mod 64 and passes its per-source sums one lane down, and the
// wavefronts of one target group take 64 / WS consecutive steps each.  After its steps a
// wavefront holds, whatever range it took, sums over its targets for every source of the block
// and sums over part of the sources for every target; both are added over the wavefronts in
// LDS in a fixed order.
//
// The sums are float64, so the split changes the rounding only in the last bits, and the tile
// is free to follow the system size: a tile pair costs 64 x 64 x (TS/64)^2 pair evaluations over
// W wavefronts, and the device needs some thousands of wavefronts.  A
// 2,100-sphere system has 15 pairs of 512-sphere tiles (one workgroup each: 120 after splitting
// the sources into parts of 64, the smallest part that still fills a rotation), but 561 of 64.
#pragma once

#include "pair_common.h"

namespace rpb {

namespace {

template <int K, bool TQ>
constexpr int sym64_rows() { return 3 * K + (TQ ? 3 : 0); }

template <int K, bool TQ, int TPT, int WT, int W>
struct Sym64Lds {
  static constexpr int kTile = 64 * WT * TPT;
  static constexpr int kStage = kTile < 64 * W ? kTile : 64 * W;   // sources staged at a time
  double x[kStage], y[kStage], z[kStage];
  double f[sym64_rows<K, TQ>()][kStage];
  // sums of a 64-source block per wavefront, two buffers (one barrier per block); the row sums
  // of the WS wavefronts of a target group go through the same memory at the end
  double col[2][W][3 * K][64];
};

// The pair of separation (dx, dy) in every vector, both directions.
template <int K, bool TQ, bool WALL>
__device__ __forceinline__ void sym64_pair(double dx, double dy, double zi, double zj,
                                           const double (&f)[sym64_rows<K, TQ>()],
                                           const double (&own)[sym64_rows<K, TQ>()],
                                           const PairConsts<double> &k, double (&acc)[3 * K],
                                           double (&cs)[3 * K]) {
  auto apply = [&](const SymCoef<double> &c) {
#pragma unroll
    for (int v = 0; v < K; ++v) {
      if constexpr (TQ && WALL) {
        if (v == 0) {
          sym_apply_both(c, f[0], f[1], f[2], own[0], own[1], own[2], f + 3 * K, own + 3 * K,
                         acc[0], acc[1], acc[2], cs[0], cs[1], cs[2]);
          continue;
        }
      }
      sym_apply<double, WALL>(c, f[3 * v], f[3 * v + 1], f[3 * v + 2], own[3 * v], own[3 * v + 1],
                              own[3 * v + 2], acc[3 * v], acc[3 * v + 1], acc[3 * v + 2],
                              cs[3 * v], cs[3 * v + 1], cs[3 * v + 2]);
    }
    if constexpr (TQ && !WALL)
      sym_apply_torque<double, WALL>(c, k, zi, f + 3 * K, own + 3 * K, acc[0], acc[1], acc[2],
                                     cs[0], cs[1], cs[2]);
  };
  const double dz = zi - zj;
  SymCoef<double> c;
  // pairs closer than 2a (rare) and the self pair take the complete form
  if (dx * dx + dy * dy + dz * dz < kFourA2) {
    sym_coefficients<double, false, TQ, WALL>(dx, dy, zi, zj, k, c);
    apply(c);
  } else {
    sym_coefficients<double, true, TQ, WALL>(dx, dy, zi, zj, k, c);
    apply(c);
  }
}

// Tile pair (I, J), I <= J, of linear index Lp: the sums of tile I's rows into slot 0 and those
// of tile J's rows into slot 1 of the pair (pm: one part per pair; a diagonal pair fills both
// slots with sums of the same rows).  On the diagonal each unordered pair is taken once, in
// 64-blocks: target block tb before source block sb in both directions, tb after sb not at all,
// and tb = sb over rotation steps 0..32 (steps 1..31 meet each pair of the block once, step 32
// meets the pairs (l, l + 32) twice and keeps lanes below 32, step 0 is the self pair, taken in
// one direction), without the steps at which a last block of few spheres has no pair (a launch of
// four vectors between two events: one sphere 17.1 -> 10.1 us, 64 spheres 16.5).  Every lane of the
// workgroup calls this (it synchronises).
template <int K, bool TQ, int TPT, int WT, int W, bool WALL, bool PERIODIC>
__device__ __forceinline__ void sym64_tile_pair(const SymArgs &a, const GeomD &g,
                                                const double *__restrict__ src,
                                                const PairConsts<double> &k,
                                                double *__restrict__ partial, const PartMap &pm,
                                                int64_t Lp, int64_t I, int64_t J,
                                                Sym64Lds<K, TQ, TPT, WT, W> &L) {
  constexpr int WS = W / WT, kSteps = 64 / WS, R = sym64_rows<K, TQ>();
  constexpr int kTile = Sym64Lds<K, TQ, TPT, WT, W>::kTile;
  constexpr int kStage = Sym64Lds<K, TQ, TPT, WT, W>::kStage;
  static_assert(WS * kTile * 3 * K <= 2 * W * 3 * K * 64 || WS == 1, "row sums fit col");
  const int tid = threadIdx.x;
  const int wave = tid / 64, lane = tid % 64;
  const int wt = wave % WT, s0 = (wave / WT) * kSteps;
  const int64_t n = a.n, first = I * kTile, jt = J * kTile;
  double tx[TPT], ty[TPT], tz[TPT], own[TPT][R], acc[TPT][3 * K];
#pragma unroll
  for (int q = 0; q < TPT; ++q) {
    const int64_t r = first + (q * WT + wt) * 64 + lane;
    const bool on = r < n;
    const int64_t i = on ? r : first;
    tx[q] = g.x[i];
    ty[q] = g.y[i];
    tz[q] = g.z[i];
#pragma unroll
    for (int e = 0; e < R; ++e) own[q][e] = on ? src[e * a.stride + r] : 0.0;
#pragma unroll
    for (int e = 0; e < 3 * K; ++e) acc[q][e] = 0.0;
  }
  const int all = int(min<int64_t>(kTile, n - jt));
  int buf = 0;
  for (int t0 = 0; t0 < all; t0 += kStage) {
    const int cnt = min(kStage, all - t0);
    if (t0 > 0) __syncthreads();
    if (tid < kStage) {   // past the last source: its position and no force
      const bool on = tid < cnt;
      const int64_t j = jt + t0 + (on ? tid : 0);
      L.x[tid] = g.x[j];
      L.y[tid] = g.y[j];
      L.z[tid] = g.z[j];
#pragma unroll
      for (int e = 0; e < R; ++e) L.f[e][tid] = on ? src[e * a.stride + j] : 0.0;
    }
    __syncthreads();
    for (int blk = 0; blk < cnt; blk += 64) {
      double cs[3 * K];   // rotating per-source sums
#pragma unroll
      for (int e = 0; e < 3 * K; ++e) cs[e] = 0.0;
      if (I != J) {
#pragma unroll(K == 1 ? 2 : 1)
        for (int s = 0; s < kSteps; ++s) {
          const int j = blk + ((lane + s0 + s) & 63);
          const double xj = L.x[j], yj = L.y[j], zj = L.z[j];
          double f[R];
#pragma unroll
          for (int e = 0; e < R; ++e) f[e] = L.f[e][j];
#pragma unroll
          for (int e = 0; e < 3 * K; ++e) cs[e] = wave_rol1(cs[e]);
#pragma unroll
          for (int q = 0; q < TPT; ++q)
            for_images<PERIODIC>(tx[q] - xj, ty[q] - yj, k, [&](double dx, double dy) {
              sym64_pair<K, TQ, WALL>(dx, dy, tz[q], zj, f, own[q], k, acc[q], cs);
            });
        }
      } else {
        const int sb = (t0 + blk) / 64;
        // No two of the block's spheres are further apart.  Held as a scalar: the batched kernels read
        // n from memory, and with a vector compare in the loop the joint batched product of 2,100
        // spheres took 190 us instead of 134.
        const int last = __builtin_amdgcn_readfirstlane(min(32, cnt - blk - 1));
#pragma unroll 1
        for (int s = 0; s < kSteps; ++s) {
          const int step = s0 + s;
          const int j = blk + ((lane + step) & 63);
          const double xj = L.x[j], yj = L.y[j], zj = L.z[j];
#pragma unroll
          for (int e = 0; e < 3 * K; ++e) cs[e] = wave_rol1(cs[e]);
#pragma unroll
          for (int q = 0; q < TPT; ++q) {
            const int tb = q * WT + wt;
            if (tb > sb || (tb == sb && step > last)) continue;   // uniform over the wavefront
            const bool fwd = tb < sb || step != 32 || lane < 32;
            const bool back = fwd && (tb < sb || step != 0);
            double f[R], o[R];
#pragma unroll
            for (int e = 0; e < R; ++e) {
              f[e] = fwd ? L.f[e][j] : 0.0;
              o[e] = back ? own[q][e] : 0.0;
            }
            for_images<PERIODIC>(tx[q] - xj, ty[q] - yj, k, [&](double dx, double dy) {
              sym64_pair<K, TQ, WALL>(dx, dy, tz[q], zj, f, o, k, acc[q], cs);
            });
          }
        }
      }
      // after step k lane l holds the sums of source (l + k) mod 64
      const int sl = (lane + s0 + kSteps - 1) & 63;
#pragma unroll
      for (int e = 0; e < 3 * K; ++e) L.col[buf][wave][e][sl] = cs[e];
      __syncthreads();
      for (int x = tid; x < 3 * K * 64; x += 64 * W) {
        const int e = x / 64, s = x % 64;
        if (blk + s < cnt) {
          double sum = 0.0;
#pragma unroll
          for (int w = 0; w < W; ++w) sum += L.col[buf][w][e][s];
          partial[part_elem(pm, Lp, 1, e / 3, e % 3, t0 + blk + s)] = sum;
        }
      }
      buf ^= 1;   // the next block's sums do not wait for this block's readers
    }
  }
  if constexpr (WS == 1) {
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int64_t local = (q * WT + wt) * 64 + lane;
      if (first + local < n)
#pragma unroll
        for (int e = 0; e < 3 * K; ++e)
          partial[part_elem(pm, Lp, 0, e / 3, e % 3, local)] = acc[q][e];
    }
  } else {
    double *rows = &L.col[0][0][0][0];   // [WS][3 K][kTile]
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TPT; ++q)
#pragma unroll
      for (int e = 0; e < 3 * K; ++e)
        rows[((wave / WT) * 3 * K + e) * kTile + (q * WT + wt) * 64 + lane] = acc[q][e];
    __syncthreads();
    for (int x = tid; x < 3 * K * kTile; x += 64 * W) {
      const int e = x / kTile, local = x % kTile;
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < WS; ++w) sum += rows[(w * 3 * K + e) * kTile + local];
      if (first + local < n) partial[part_elem(pm, Lp, 0, e / 3, e % 3, local)] = sum;
    }
  }
}

// One workgroup per tile pair of the chunk [pm.L0, pm.L0 + gridDim.x).
template <int K, bool TQ, int TPT, int WT, int W, bool WALL, bool PERIODIC>
__global__ __launch_bounds__(64 * W) void pair_kernel_f64_tiles(SymArgs a, PartMap pm, GeomD g,
                                                                const double *__restrict__ src,
                                                                PairConsts<double> k,
                                                                double *__restrict__ partial) {
  if (a.skip && *a.skip) return;
  __shared__ Sym64Lds<K, TQ, TPT, WT, W> L;
  int64_t I, J;
  const int64_t Lp = pm.L0 + int64_t(blockIdx.x);
  tri_decode(Lp, a.nt, I, J);
  sym64_tile_pair<K, TQ, TPT, WT, W, WALL, PERIODIC>(a, g, src, k, partial, pm, Lp, I, J, L);
}

}  // namespace

}  // namespace rpb
