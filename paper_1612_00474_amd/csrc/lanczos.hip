// Krylov/Lanczos approximation of M^{1/2} w (paper, Sec. II.C, method of Ando et al.).
//
// Everything but the O(N^2) products is float64 and O(N m):
//   v_1 = w/|w|;  for m = 1, 2, ...:
//     u = M v_m;  alpha_m = v_m . u;  u -= alpha_m v_m + beta_{m-1} v_{m-1};
//     u -= V_m (V_m^T u)                       (full re-orthogonalisation)
//     beta_m = |u|
//     y_m = |w| T_m^{1/2} e_1    (quadrature, or T_m = Q L Q^T updated from T_{m-1}'s)
//     eps_m = |y_m - (y_{m-1}, 0)| / |y_{m-1}|  (= |g_m - g_{m-1}|/|g_{m-1}| for orthonormal V)
//     stop if eps_m < tol (m >= 2), or beta_m ~ 0 (invariant Krylov space, exact result)
//     v_{m+1} = u / beta_m
//   g = V_m y_m.
// Reductions use a fixed number of blocks and a fixed tree, so results are bitwise
// reproducible.  Each iteration's stop test is tagged into pinned memory, which the host polls.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstddef>
#include <type_traits>
#include <vector>

#include "pair_common.h"
#include "rpb_internal.h"

namespace rpb {

namespace {

constexpr int kMaxKrylov = 64;      // largest m (the eigensolve keeps T_m in one wavefront)
constexpr int kThreads = 256;

// Device-side Lanczos scalars (lives at the start of the WS_SMALL slot).
struct LzState {
  double alpha[kMaxKrylov];
  double beta[kMaxKrylov];
  double y[kMaxKrylov];
  double yprev[kMaxKrylov];
  double wnorm;
  int eig_m;      // order of the eigendecomposition held in LzEig (0: none)
  int pad_;
  // status (read by the host every iteration)
  double eps;
  int m;
  int reason;     // 0 running, 1 converged, 2 breakdown, 3 not SPD, 4 eigensolve failed
};
static_assert(sizeof(LzState) % 8 == 0, "LzState is an array of doubles and pairs of ints");
static_assert(sizeof(LzState) <= kSmallWorkCounter, "LzState must fit the start of the small slot");
static_assert(size_t(kMaxBatchSystems) * sizeof(LzStatus) <= kHostLzRingOffset,
              "per-system records must stay below the status ring");

// Host copies of the status words of consecutive iterations, slot k mod kLzRing for iteration k.
// The kernel that ends an iteration's stop test stores them and then the tag that the host waits
// for (an event after the kernel would cost the device ~5 us per iteration).
struct LzRingSlot {
  double eps;
  int reason;
  int tag;
};
struct LzRing {
  LzRingSlot slot[kLzRing];
};

LzRing *lz_ring(rpb_ctx *ctx) {
  return reinterpret_cast<LzRing *>(static_cast<char *>(host_scratch(ctx)) + kHostLzRingOffset);
}
// The ring as kernels address it.
LzRing *lz_ring_dev(rpb_ctx *ctx) {
  return reinterpret_cast<LzRing *>(static_cast<char *>(host_scratch_dev(ctx)) +
                                    kHostLzRingOffset);
}

// Tags of a solve: its epoch (from 1, unique in the context until it wraps after 2^23 solves, whose
// pinned buffer starts zeroed), the iteration and, for the processes of a batch, a stop bit.
constexpr int kTagStop = 0x80;
__host__ __device__ __forceinline__ int lz_tag(int epoch, int k) { return (epoch << 8) | k; }
int next_epoch(rpb_ctx *ctx) {
  ctx->lz_epoch = ctx->lz_epoch >= 0x7fffff ? 1 : ctx->lz_epoch + 1;
  return ctx->lz_epoch;
}

// out = V y (first nvec rows of V)
__global__ void basis_combine(int64_t m, int nvec, const double *__restrict__ V,
                              const double *__restrict__ y, double *__restrict__ out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= m) return;
  double acc = 0.0;
  for (int k = 0; k < nvec; ++k) acc += y[k] * V[int64_t(k) * m + i];
  out[i] = acc;
}

// Orders a wavefront's own accesses before its later accesses to other lanes' words.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Eigendecomposition of T_m kept from one order to the next (the eigensolve of T_{m+1} updates
// it): eigenvalues in increasing order and the eigenvector matrix of T_m, column-major.
struct LzEig {
  double lam[kMaxKrylov];
  double Q[kMaxKrylov * kMaxKrylov];   // Q[col * kMaxKrylov + row]
};

// LDS of the root of T_m: the quadrature's transposed sums or the arrowhead's eigenvectors.
constexpr int kRootPool = 4 * 16 * 65;
static_assert(kRootPool >= kMaxKrylov * kMaxKrylov, "the eigenvectors fit the pool");

// 1/x: the hardware estimate refined by two Newton steps r <- r + r (1 - x r) (the error is
// squared by each; the result is within an ulp or two of the rounded quotient), about half the
// instructions of an IEEE division.  x finite and nonzero.
__device__ __forceinline__ double rcp_f64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}

constexpr int kMaxRootIter = 64;   // secular-equation iterations per root before giving up

// The p + 1 roots of the secular equation of an arrowhead matrix with diagonal d (p distinct
// values, increasing), border z (no zero; z2 = z^2) and corner a:
//   f(mu) = a - mu - sum_j z_j^2 / (d_j - mu),
// decreasing between consecutive poles, so that root i lies in (d_{i-1}, d_i) (d_{-1} = -inf,
// d_p = +inf; the outer roots lie within |z| of d or a).  Root i is kept as mu = d_K + tau about
// its nearer pole K (the sign of f at the midpoint of the interval decides), with d_j - mu
// formed as (d_j - d_K) - tau, so that it keeps full relative accuracy in its distance to the
// pole.  Each step solves the model c + b tau + z_K^2 / tau = 0 (the pole K exact, the other
// terms linearised at the current tau: a quadratic with one root on each side of 0, the one on
// the side of the root is taken), safeguarded by bisection of the bracket; a root stops when
// |f| is within the rounding error of its terms, or when a step no longer moves it.
// Lane i of every wavefront follows root i; wavefront w sums the terms j = w, w + W, ... and
// the W partial sums are added in wavefront order through LDS, so every wavefront holds the
// same totals and takes the same steps.  Every thread of the workgroup calls this (W <=
// kThreads / 64); wavefront 0 writes K, tau, d_K and a failure flag (no stop within
// kMaxRootIter steps) for each root (K = -1, tau = 0 when p = 0: the root is a itself).
__device__ void secular_roots(int p, const double *__restrict__ d, const double *__restrict__ z2,
                              double a, int *K_out, double *tau_out, double *dK_out,
                              int *fail_out) {
  constexpr int kMaxW = kThreads / 64;
  __shared__ double part[2][kMaxW][4][64];
  __shared__ int more_s[2][kMaxW];
  const int w = int(threadIdx.x) / 64, i = int(threadIdx.x) & 63;
  // the terms are split over the wavefronts only when there are enough of them to pay for
  // the exchange (one barrier per step); otherwise the first wavefront takes them all
  const int W = p >= 16 ? kMaxW : 1;
  if (w >= W) return;   // wavefront-uniform; the caller's next barrier joins them again
  const bool act = p > 0 && i <= p;
  int buf = 0;
  // sums over all terms of w_j, |w_j|, and, without j = K, of w_j and w_j / (d_j - mu), with
  // w_j = z_j^2 / ((d_j - x0) - x1); with W > 1 also whether any wavefront reports `need`
  auto sums = [&](double x0, double x1, int K, bool need, double (&tot)[4]) -> bool {
    const bool any = __ballot(need) != 0ull;
    if (W == 1 && !any) return false;   // alone, the wavefront stops before summing again
    double f = 0.0, mag = 0.0, R = 0.0, Rp = 0.0;
    auto term = [&](int j, double inv) {
      const double t = z2[j] * inv;
      f += t;
      mag += fabs(t);
      if (j != K) {
        R += t;
        Rp += t * inv;
      }
    };
    if (act) {
      // four reciprocals in flight at a time; the sums still run in increasing j
      int j = w;
      for (; j + 3 * W < p; j += 4 * W) {
        double inv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) inv[r] = rcp_f64((d[j + r * W] - x0) - x1);
#pragma unroll
        for (int r = 0; r < 4; ++r) term(j + r * W, inv[r]);
      }
      for (; j < p; j += W) term(j, rcp_f64((d[j] - x0) - x1));
    }
    if (W == 1) {
      tot[0] = f;
      tot[1] = mag;
      tot[2] = R;
      tot[3] = Rp;
      return any;
    }
    part[buf][w][0][i] = f;
    part[buf][w][1][i] = mag;
    part[buf][w][2][i] = R;
    part[buf][w][3][i] = Rp;
    if (i == 0) more_s[buf][w] = any ? 1 : 0;
    __syncthreads();
    bool more = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double v = part[buf][0][q][i];
      for (int u = 1; u < W; ++u) v += part[buf][u][q][i];
      tot[q] = v;
    }
    for (int u = 0; u < W; ++u) more = more || more_s[buf][u] != 0;
    buf ^= 1;   // the next exchange uses the other buffer, so no second barrier is needed
    return more;
  };
  double zn2 = 0.0;
#pragma unroll 4
  for (int j = 0; j < p; ++j) zn2 += z2[j];
  const double znorm = sqrt(zn2);
  // bracket and pole of every root, and the first evaluation: an interior root at the midpoint
  // of its two poles (every term: the sign of f there picks the pole), an outer root half way
  // into its bracket about its only pole
  int K = 0;
  double lo = 0.0, hi = 0.0, x0 = 0.0, x1 = 0.0;
  if (act) {
    if (i == 0) {
      K = 0;
      lo = fmin(d[0], a) - znorm - d[0];
      x0 = d[0];
      x1 = 0.5 * lo;
    } else if (i == p) {
      K = p - 1;
      hi = fmax(d[p - 1], a) + znorm - d[p - 1];
      x0 = d[p - 1];
      x1 = 0.5 * hi;
    } else {
      K = -1;
      x0 = 0.5 * (d[i - 1] + d[i]);
    }
  }
  double tot[4];
  sums(x0, x1, K, true, tot);
  double tau = x1;
  if (act && i > 0 && i < p) {
    const double mid = x0;
    if ((a - mid) - tot[0] > 0.0) {   // the root lies above the midpoint: pole d_i
      K = i;
      lo = mid - d[i];
      tau = lo;
    } else {
      K = i - 1;
      hi = mid - d[i - 1];
      tau = hi;
    }
    // the sums without pole K, from those over every term
    const double inv = 1.0 / (d[K] - mid), t = z2[K] * inv;
    tot[2] -= t;
    tot[3] -= t * inv;
  }
  const double dK = act ? d[K] : 0.0, a0 = a - dK, zK2 = act ? z2[K] : 0.0;
  const bool above = K == i - 1;   // the root lies above its pole (tau > 0)
  bool done = !act, ok = !act;
  // every wavefront of the exchange sees the same `more`, so all take the same number of steps
  for (int it = 0; it == 0 || sums(dK, tau, K, !done, tot); ++it) {
    if (done) continue;
    const double f = (a0 - tau) - tot[0];
    const double mag = (fabs(a0) + fabs(tau)) + tot[1];
    if (fabs(f) <= 4.0 * DBL_EPSILON * mag) {
      done = ok = true;
      continue;
    }
    if (f > 0.0)
      lo = tau;
    else
      hi = tau;
    const double b = -1.0 - tot[3];           // slope of the linearised part
    const double c = (a0 - tau - tot[2]) - b * tau;
    const double disc = sqrt(c * c - 4.0 * b * zK2);
    // the quadratic's root on the side of the pole, in the form without cancellation
    const bool neg = c <= 0.0;
    const double num = above ? (neg ? 2.0 * zK2 : c + disc) : (neg ? disc - c : 2.0 * zK2);
    const double den = above ? (neg ? disc - c : -2.0 * b) : (neg ? 2.0 * b : -c - disc);
    double t = num * rcp_f64(den);
    if (!(t >= lo && t <= hi)) t = 0.5 * (lo + hi);
    if (fabs(t - tau) <= 2.0 * DBL_EPSILON * fabs(t)) done = ok = true;
    tau = t;
    if (it + 1 >= kMaxRootIter) done = true;
  }
  if (w == 0 && i <= p) {
    K_out[i] = act ? K : -1;
    tau_out[i] = act ? tau : 0.0;
    dK_out[i] = act ? dK : 0.0;
    fail_out[i] = ok ? 0 : 1;
  }
}

// Eigendecomposition of T_m from that of T_{m-1} (in eig, replaced by T_m's), for the T_m that
// root_quadrature does not take.  In the basis of
// T_{m-1}'s eigenvectors and e_m, T_m is an arrowhead matrix: diagonal lambda, border
// z = beta_{m-1} (last row of Q), corner alpha_m.  Its eigenproblem is solved as in the
// divide-and-conquer method (Cuppen 1981; Gu and Eisenstat 1995):
//   - deflation: a border entry below tol (8 eps |T|) leaves its lambda an eigenvalue; two
//     lambdas closer than tol / (c s) are rotated so that one border entry vanishes;
//   - the p + 1 roots of the secular equation of the rest, one lane each (secular_root);
//   - a border recomputed from the roots, z^_j^2 = prod_i |d_j - mu_i| / prod_{l != j}
//     |d_j - d_l| (the border for which the computed roots are exact), which keeps the
//     eigenvectors u_i = (z^_j / (d_j - mu_i), -1) / norm orthogonal to working accuracy;
//   - new eigenvectors [Q 0; 0 1] U and the eigenvalues sorted increasingly.
// Every thread of the workgroup calls this; the first wavefront (one lane per eigenvalue, m <=
// 64) does the scalar work and the workgroup forms the product.  Returns 1 (every thread)
// when a root iteration did not stop or an eigenvalue is not finite.
__device__ int eig_update(int m, const LzState *__restrict__ st, LzEig *__restrict__ eig,
                          double *__restrict__ U) {
  // column-major (entry [row or component] fastest), so that the lanes of a wavefront, which
  // take consecutive rows, touch consecutive words; U (LDS, kRootPool): eigenvectors of the
  // arrowhead, [j * 64 + i].  Q is rotated and then replaced in place.
  double *Q = eig->Q;
  __shared__ double dd[kMaxKrylov], zz[kMaxKrylov], dn[kMaxKrylov], z2n[kMaxKrylov];
  __shared__ double zh[kMaxKrylov], tau_s[kMaxKrylov], dK_s[kMaxKrylov], val[kMaxKrylov];
  __shared__ double rot_c[kMaxKrylov], rot_s[kMaxKrylov];
  __shared__ int K_s[kMaxKrylov], nd_s[kMaxKrylov], df_s[kMaxKrylov], rank_s[kMaxKrylov];
  __shared__ int fail_s[kMaxKrylov];
  __shared__ int rot_p[kMaxKrylov], rot_j[kMaxKrylov];
  __shared__ int info[4];   // p, number of deflated, number of rotations, failure
  const int tid = threadIdx.x, nthr = kThreads;
  const int lane = tid & 63;
  const bool w0 = tid < 64;
  if (m == 1) {
    if (tid == 0) {
      eig->lam[0] = st->alpha[0];
      Q[0] = 1.0;
    }
    __syncthreads();
    return 0;
  }
  const int n1 = m - 1;
  const double alpha = st->alpha[m - 1], beta = st->beta[m - 2];
  if (w0) {
    if (lane < n1) {
      dd[lane] = eig->lam[lane];
      zz[lane] = beta * Q[lane * kMaxKrylov + (n1 - 1)];
    }
    // deflation tolerance from |T_m| <= max(|lambda|, |alpha|) + |beta|
    double amax = lane < n1 ? fabs(eig->lam[lane]) : 0.0;
    for (int off = 32; off > 0; off >>= 1) amax = fmax(amax, __shfl_xor(amax, off, 64));
    const double tol = 8.0 * DBL_EPSILON * (fmax(amax, fabs(alpha)) + fabs(beta));
    // the wavefront's LDS accesses complete in order: dd and zz are visible below
    const double zj = lane < n1 ? zz[lane] : 0.0;
    unsigned long long keep = __ballot(lane < n1 && fabs(zj) > tol);
    // a kept entry and the kept entry before it that would rotate into one (parallel test;
    // the rotations themselves are taken in order, below, only when some pair qualifies)
    bool close = false;
    if ((keep >> lane) & 1ull) {
      const unsigned long long below = keep & ((1ull << lane) - 1ull);
      if (below) {
        const int q = 63 - __builtin_clzll(below);
        const double zq = zz[q], r = sqrt(zq * zq + zj * zj);
        close = fabs((zj / r) * (zq / r) * (dd[lane] - dd[q])) <= tol;
      }
    }
    int nrot = 0;
    if (__ballot(close)) {
      // in order over the entries, every lane alike: a kept entry q followed by a kept j
      // whose rotation deflates q
      keep = 0;
      int prev = -1;
      for (int j = 0; j < n1; ++j) {
        const double zjj = zz[j];
        if (!(fabs(zjj) > tol)) continue;
        if (prev >= 0) {
          const double zp = zz[prev], r = sqrt(zp * zp + zjj * zjj);
          const double c = zjj / r, sn = zp / r;
          if (fabs(c * sn * (dd[j] - dd[prev])) <= tol) {
            const double dp = dd[prev], dj = dd[j];
            if (lane == 0) {
              dd[prev] = c * c * dp + sn * sn * dj;
              dd[j] = sn * sn * dp + c * c * dj;
              zz[prev] = 0.0;
              zz[j] = r;
              rot_p[nrot] = prev;
              rot_j[nrot] = j;
              rot_c[nrot] = c;
              rot_s[nrot] = sn;
            }
            ++nrot;
            keep &= ~(1ull << prev);
          }
        }
        keep |= 1ull << j;
        prev = j;
      }
    }
    const int p = __popcll(keep);
    const unsigned long long lower = (1ull << lane) - 1ull;
    if (lane < n1) {
      if ((keep >> lane) & 1ull) {
        const int q = __popcll(keep & lower);
        dn[q] = dd[lane];
        z2n[q] = zz[lane] * zz[lane];
        nd_s[q] = lane;
      } else {
        df_s[__popcll(~keep & lower)] = lane;
      }
    }
    if (lane == 0) {
      info[0] = p;
      info[1] = n1 - p;
      info[2] = nrot;
    }
  }
  __syncthreads();
  const int p = info[0], ndf = info[1], nrot = info[2];
  // the deflating rotations on the columns of the old Q, in order
  for (int q = 0; q < nrot; ++q) {
    const int a = rot_p[q], b = rot_j[q];
    const double c = rot_c[q], sn = rot_s[q];
    for (int r = tid; r < n1; r += nthr) {
      const double qa = Q[a * 64 + r], qb = Q[b * 64 + r];
      Q[a * 64 + r] = c * qa - sn * qb;
      Q[b * 64 + r] = sn * qa + c * qb;
    }
    __syncthreads();
  }
  // the roots (with p = 0 the arrowhead is alpha alone), by the whole workgroup
  secular_roots(p, dn, z2n, alpha, K_s, tau_s, dK_s, fail_s);
  if (w0) {
    int bad = 0;
    if (lane <= p) {
      bad = fail_s[lane];
      const int K = K_s[lane];
      val[lane] = K >= 0 ? dK_s[lane] + tau_s[lane] : alpha;
    } else if (lane < m) {
      val[lane] = dd[df_s[lane - p - 1]];
    }
    // the recomputed border: the numerator's roots paired with the denominator's poles
    if (lane < p) {
      const double dj = dn[lane];
      // each factor formed apart from the running product, so that only a multiply waits on it
      double prod = 1.0;
#pragma unroll 4
      for (int i = 0; i <= p; ++i) {
        const double num = fabs((dj - dK_s[i]) - tau_s[i]);
        prod *= (i < p && i != lane) ? num * rcp_f64(fabs(dj - dn[i])) : num;
      }
      zh[lane] = sqrt(prod);   // its sign: that of the border entry, which z2n does not keep
      const double zs = zz[nd_s[lane]];
      if (zs < 0.0) zh[lane] = -zh[lane];
    }
    // eigenvector lane of the arrowhead (entries 0..p-1 on the kept lambdas, p on e_m)
    if (lane <= p) {
      double nrm = 1.0;
      if (p > 0) {
        const int K = K_s[lane];
        const double dK = dn[K], tau = tau_s[lane];
#pragma unroll 4
        for (int j = 0; j < p; ++j) {
          const double x = zh[j] * rcp_f64((dn[j] - dK) - tau);
          U[j * 64 + lane] = x;
          nrm += x * x;
        }
      }
      const double inv = 1.0 / sqrt(nrm);
#pragma unroll 4
      for (int j = 0; j < p; ++j) U[j * 64 + lane] *= inv;
      U[p * 64 + lane] = -inv;
    }
    // rank of every eigenvalue (ties by index)
    if (lane < m) {
      const double v = val[lane];
      int r = 0;
#pragma unroll 8
      for (int e = 0; e < m; ++e) {
        const double ve = val[e];
        r += (ve < v || (ve == v && e < lane)) ? 1 : 0;
      }
      rank_s[lane] = r;
      eig->lam[r] = v;
      bad |= !isfinite(v);
    }
    bad = __ballot(bad) != 0ull;
    if (lane == 0) info[3] = bad;
  }
  __syncthreads();
  // new eigenvectors: column rank(e) of Q_m, rows 0..m-1.  A row of the new Q needs the same row of
  // the old one only, so a wavefront takes a row (lane e its entry e) and overwrites it.
  for (int r = tid >> 6; r < m; r += nthr / 64) {
    const int e = lane;
    double v = 0.0;
    if (e <= p) {
      if (r < n1) {
        // four running sums keep several loads in flight
        double v4[4] = {0.0, 0.0, 0.0, 0.0};
        int j = 0;
        for (; j + 4 <= p; j += 4)
#pragma unroll
          for (int q = 0; q < 4; ++q) v4[q] += Q[nd_s[j + q] * 64 + r] * U[(j + q) * 64 + e];
        for (; j < p; ++j) v4[0] += Q[nd_s[j] * 64 + r] * U[j * 64 + e];
        v = (v4[0] + v4[1]) + (v4[2] + v4[3]);
      } else {
        v = U[p * 64 + e];
      }
    } else if (e < m && r < n1) {
      v = Q[df_s[e - p - 1] * 64 + r];
    }
    wave_sync();
    if (e < m) Q[rank_s[e] * kMaxKrylov + r] = v;
  }
  __syncthreads();
  return info[3];
}

// T^{1/2} e_1 without an eigendecomposition, from T^{1/2} = (2/pi) int_0^inf T (T + t^2)^{-1} dt with
// t = e^x: the trapezoidal rule converges as exp(-pi^2/h) (the integrand's poles lie at
// distance pi/2 from the real axis), 4e-22 at h = 0.2.  Thread k takes node t_k = sqrt(G) e^{(k -
// 191.5) h}, G >= |T| by Gershgorin, and solves (T + t_k^2) x = e_1 by elimination from the last
// row; the solutions are independent chains of m reciprocals.  Nodes below sqrt(G) add t (e_1 -
// t^2 x) and the others t T x (neither form cancels by more than |T|^{1/2}); what lies below t_0
// and above t_255 is summed as the geometric series it has become to (t_0^2/lambda_min and
// |T|/t_255^2 cubed roots of 1e-16).  The error is that of T^{1/2} under a rounding of T,
// ~eps (|T|/lambda_min)^{1/2} |T|^{1/2}, as with an eigendecomposition.
// A pivot of T itself below 1e-8 G (T indefinite, singular or nearly so) or a value that is not
// finite returns 0 on every thread and the caller takes the eigendecomposition.  Else lane r of
// the first wavefront returns row r of T^{1/2} e_1 in y.
// One chain of m dependent steps instead of the root searches and the product of the updated
// eigendecomposition: lanczos_eig over m = 1..26 16.7 -> 6.4 us, beta_eig over m = 1..12 (which
// also sums beta) 13.2 -> 7.3 us; the 2,100-sphere step 714 -> 677 us.
constexpr double kRootStep = 0.2;
constexpr int kRootLow = 192;   // nodes below sqrt(G): the first three wavefronts

struct RootLds {
  double a[kMaxKrylov], b[kMaxKrylov], b2[kMaxKrylov];
  double sum[kThreads / 64][kMaxKrylov];   // per wavefront: sum over its nodes of c x_i
  double z[kMaxKrylov + 2];                // padded, z[i + 1]
  int ok;
};

// The weighted solutions of this thread's node for the leading M rows (rows past m are decoupled),
// summed over each wavefront into L.sum.
template <int M>
__device__ __forceinline__ void root_nodes(double G, RootLds &L, double *__restrict__ pool) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const double node = sqrt(G) * exp((double(t) - (kRootLow - 0.5)) * kRootStep);
  const double sh = node * node;
  const double cw = t < kRootLow ? node * sh : node;
  double r[M];
  const double floor_ = 1e-8 * G;
  double d = L.a[M - 1] + sh;
  bool ok = d >= floor_;
  r[M - 1] = rcp_f64(d);
#pragma unroll
  for (int i = M - 2; i >= 0; --i) {
    d = (L.a[i] + sh) - L.b2[i] * r[i + 1];
    ok = ok && d >= floor_;
    r[i] = rcp_f64(d);
  }
  if (t == 0) L.ok = ok && isfinite(r[0]);   // the smallest shift: the pivots of T
  double x = r[0] * cw;
  r[0] = x;
#pragma unroll
  for (int i = 1; i < M; ++i) {
    x *= -L.b[i - 1] * r[i];
    r[i] = x;
  }
  // 16 rows at a time: transposed through LDS, four lanes per row add 16 nodes each
  double *p = pool + wave * 16 * 65;
#pragma unroll
  for (int i0 = 0; i0 < M; i0 += 16) {
    constexpr int R = M < 16 ? M : 16;
#pragma unroll
    for (int i = 0; i < R; ++i) p[i * 65 + lane] = r[i0 + i];
    wave_sync();
    const int row = lane >> 2, q = lane & 3;
    double v = 0.0;
    if (row < R)
#pragma unroll
      for (int j = 0; j < 16; ++j) v += p[row * 65 + q * 16 + j];
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    if (q == 0 && row < R) L.sum[wave][i0 + row] = v;
    wave_sync();
  }
}

__device__ int root_quadrature(int m, const LzState *__restrict__ st, RootLds &L,
                               double *__restrict__ pool, double &y) {
  const int t = threadIdx.x, lane = t & 63;
  const double ai = lane < m ? st->alpha[lane] : 0.0;
  const double bi = lane < m - 1 ? st->beta[lane] : 0.0;
  const double bp = __shfl_up(bi, 1, 64);
  double G = fabs(ai) + fabs(bi) + (lane > 0 ? fabs(bp) : 0.0);
  for (int off = 32; off > 0; off >>= 1) G = fmax(G, __shfl_xor(G, off, 64));
  if (!(G > 1e-100 && G < 1e100)) return 0;   // the same on every thread; t^3 stays in range
  if (t < 64) {
    L.a[lane] = lane < m ? ai : G;
    L.b[lane] = bi;
    L.b2[lane] = bi * bi;
  }
  __syncthreads();
  if (m <= 8)
    root_nodes<8>(G, L, pool);
  else if (m <= 16)
    root_nodes<16>(G, L, pool);
  else if (m <= 32)
    root_nodes<32>(G, L, pool);
  else
    root_nodes<64>(G, L, pool);
  __syncthreads();
  if (!L.ok) return 0;
  if (t < 64) {
    const double eh = exp(-kRootStep), tail = 1.0 / (1.0 - eh), sG = sqrt(G);
    // sum of every node below sqrt(G) down to 0, and of 1/t beyond the last node
    const double low = sG * exp(-0.5 * kRootStep) * tail;
    const double high = tail * exp(-(kThreads - kRootLow + 0.5) * kRootStep) / sG;
    const double A = (L.sum[0][lane] + L.sum[1][lane]) + L.sum[2][lane];
    const double B = L.sum[3][lane] + (lane == 0 ? high : 0.0);
    const double z = lane < m ? B : 0.0;
    L.z[lane + 1] = z;
    if (lane == 0) L.z[0] = L.z[kMaxKrylov + 1] = 0.0;
    wave_sync();
    const double Tz = (lane > 0 ? L.b[lane - 1] * L.z[lane] : 0.0) + ai * z +
                      (lane < m - 1 ? bi * L.z[lane + 2] : 0.0);
    y = (2.0 * kRootStep / M_PI) * (((lane == 0 ? low : 0.0) - A) + Tz);
  }
  return 1;
}

// y_m = |w| T_m^{1/2} e_1 (root_quadrature, or the eigendecomposition of T_m brought up from the
// order it was left at, negative eigenvalues taken as zero), eps_m and the stop test.  Every
// thread of the workgroup (kThreads) calls this; the first wavefront forms y_m and the status.
__device__ void tridiag_body(int m, double tol, LzState *__restrict__ st, LzEig *__restrict__ eig) {
  static_assert(kThreads == 256, "one quadrature node per thread");
  __shared__ RootLds L;
  __shared__ double pool[kRootPool];
  __shared__ double Rz[kMaxKrylov];   // sqrt(lambda_k) q_k[0]
  double yr = 0.0;
  // The pivots from the last row (the first entry of each trailing block's inverse) never grow with
  // m and the bound on |T| never falls, so a T_m whose predecessor was left to the
  // eigendecomposition is left to it too.
  const bool left = m > 1 && st->eig_m == m - 1;
  const int fast = left ? 0 : root_quadrature(m, st, L, pool, yr);
  int failed = 0;
  bool indefinite = false;
  const int lane = threadIdx.x;
  if (!fast) {
    const int have = st->eig_m;
    __syncthreads();   // every thread has read eig_m and is done with the pool
    for (int k = have + 1; k <= m; ++k) {
      failed |= eig_update(k, st, eig, pool);
      __syncthreads();
    }
    if (lane < 64) {
      const double *Q = eig->Q;
      const double lmin = eig->lam[0], lmax = eig->lam[m - 1];
      indefinite = lmin < -1e-12 * fmax(lmax, 0.0);
      // lane k forms sqrt(lambda_k) q_k[0], then lane r sums row r
      if (lane < m) Rz[lane] = sqrt(fmax(eig->lam[lane], 0.0)) * Q[lane * kMaxKrylov];
      yr = 0.0;
      if (lane < m) {
#pragma unroll 4
        for (int k = 0; k < m; ++k) yr += Rz[k] * Q[k * kMaxKrylov + lane];
      }
      if (lane == 0) st->eig_m = m;
    }
  }
  if (lane >= 64) return;
  double amax = lane < m ? fabs(st->alpha[lane]) : 0.0;
  for (int off = 32; off > 0; off >>= 1) amax = fmax(amax, __shfl_xor(amax, off, 64));
  yr = lane < m ? yr * st->wnorm : 0.0;
  // eps_m in the orthonormal Krylov basis
  const double yp = (lane < m - 1) ? st->yprev[lane] : 0.0;
  const double diff = (lane < m) ? (yr - yp) : 0.0;
  double num = diff * diff, den = yp * yp;
  for (int off = 32; off > 0; off >>= 1) {
    num += __shfl_xor(num, off, 64);
    den += __shfl_xor(den, off, 64);
  }
  if (lane < m) {
    st->y[lane] = yr;
    st->yprev[lane] = yr;
  }
  if (lane == 0) {
    const double eps = m >= 2 ? sqrt(num / den) : 0.0;
    int reason = 0;
    if (failed)
      reason = 4;
    else if (indefinite)
      reason = 3;
    else if (m >= 2 && eps < tol)
      reason = 1;
    else if (st->beta[m - 1] <= 1e-14 * amax)
      reason = 2;
    st->eps = eps;
    st->m = m;
    st->reason = reason;
  }
}

// Status words of iteration k into the host's ring slot, by one thread after the state is final; the
// release orders the tag after the two words before it.
__device__ __forceinline__ void post_status(const LzState *__restrict__ st, LzRingSlot *slot,
                                            int tag) {
  slot->eps = st->eps;
  slot->reason = st->reason;
  __hip_atomic_store(&slot->tag, tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- Krylov processes on segments of concatenated vectors -------------------------------------
//
// Process s owns elements [3 offs[s], 3 offs[s + 1]) of every vector (offs NULL: one process, all
// m3 elements) and its own LzState.  done[s] != 0 (done NULL for a single process) freezes a
// process: every kernel skips it, so it stops changing once its own tolerance or breakdown test
// is met, whatever the others do.
//
// After the product u = M v_k, an iteration is two kernels, and the sum alpha_k = v_k . u is taken
// with the product's own reduction, one partial per 64 rows:
//   lz_dots    u <- u - alpha_k v_k - beta_{k-1} v_{k-1} (every workgroup sums the partials of
//              alpha), h_j = V_j . u for j <= k and |u|^2, one partial per workgroup; each
//              workgroup keeps its elements in registers over all basis vectors;
//   lz_update  every workgroup sums h and |u|^2, so beta_k^2 = |u - V_k h|^2 = |u|^2 - |h|^2 (the h_j
//              are rounding errors, so nothing cancels unless the Krylov space is exhausted, where
//              beta_k is a rounding error either way) needs no third pass, and
//              v_{k+1} = (u - V_k h) / beta_k goes to the basis and, weighted, into the next
//              product's sources; the process's first workgroup then takes T_k^{1/2} e_1 and the
//              stop test.
// The work is a few reads of vectors that fit the caches; what bounds it is the ~4.4 us that each
// dependent launch costs, so the count is what matters: six kernels per iteration before (two
// for alpha, dots, their sum, update, beta and root, scaling), 93 -> 38 us per iteration at 2,100
// spheres, product included (92 -> 67 with a mixed product, whose vector work has four kernels).

constexpr int kPartRows = 64;   // rows per partial of alpha

struct SegView {
  const int64_t *offs;    // nsys + 1 (device); NULL: one process
  const int *sys_of;      // sphere -> system (device)
  LzState *st;            // nsys states
  int *done;              // nsys flags, the all-done flag, the count of finished processes
  LzEig *eig;             // nsys eigendecompositions
  int nsys;
  int64_t m3;             // elements of a vector
  // workgroups of kThreads and of 4 kThreads values (BlockList's lists, nullable)
  const int2 *list1, *list4;
};

__device__ __forceinline__ void seg_range(const SegView &v, int s, int64_t &e0, int64_t &e1) {
  e0 = v.offs ? 3 * v.offs[s] : 0;
  e1 = v.offs ? 3 * v.offs[s + 1] : v.m3;
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum of np partials by the whole workgroup, the same value on every thread (sh: kThreads / 64).
__device__ __forceinline__ double sum_partials(const double *__restrict__ part, int64_t np,
                                               double *sh) {
  double a = 0.0;
  for (int64_t i = threadIdx.x; i < np; i += kThreads) a += part[i];
  a = wave_sum(a);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  double r = sh[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) r += sh[w];
  __syncthreads();
  return r;
}

// The workgroup's process and its place among the process's workgroups of EPT kThreads values.
template <int EPT>
__device__ __forceinline__ void seg_block(const SegView &v, int &s, int &blk) {
  static_assert(EPT == 1 || EPT == 4, "lists of these");
  block_of(EPT == 1 ? v.list1 : v.list4, s, blk);
}

// One partial per 64 elements of a . b over each live process (workgroups of kThreads values);
// partials of process s from part[first_partial(its first element, s, kPartRows)].
__global__ __launch_bounds__(kThreads) void lz_dot(SegView v, const double *__restrict__ a,
                                                   const double *__restrict__ b, int check_done,
                                                   double *__restrict__ part) {
  int s, blk;
  seg_block<1>(v, s, blk);
  if (check_done && v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  const int64_t i = e0 + int64_t(blk) * kThreads + threadIdx.x;
  const double x = wave_sum(i < e1 ? a[i] * b[i] : 0.0);
  const int64_t q = int64_t(blk) * (kThreads / 64) + (threadIdx.x >> 6);
  if ((threadIdx.x & 63) == 0 && e0 + q * kPartRows < e1)
    part[first_partial(e0, s, kPartRows) + q] = x;
}

// The state of process s at its start, by one workgroup.
__device__ __forceinline__ void reset_state(const SegView &v, int s, double wn) {
  LzState *st = v.st + s;
  const int t = threadIdx.x;
  if (t < kMaxKrylov) st->alpha[t] = st->beta[t] = st->y[t] = st->yprev[t] = 0.0;
  if (t == 0) {
    st->wnorm = wn;
    st->eig_m = 0;
    st->eps = 0.0;
    st->m = 0;
    st->reason = 0;
    if (v.done) v.done[s] = 0;
  }
}

// Start of every process: |w| from the partials of w . w, the state reset, v_1 = w / |w| into the
// basis and, with src, into the first product's packed sources; with mw = M w also u = mw / |w| and
// the partials of alpha_1 = v_1 . u.  counter (nullable): a persistent kernel's work counter, zeroed.
template <typename Real>
__global__ __launch_bounds__(kThreads) void lz_start(
    SegView v, const double *__restrict__ w, const double *__restrict__ npart,
    double *__restrict__ V, const double *__restrict__ hw, Real *__restrict__ src,
    const double *__restrict__ mw, double *__restrict__ u, double *__restrict__ apart,
    int *counter) {
  __shared__ double sh[kThreads / 64];
  const int t = threadIdx.x;
  int s, blk;
  seg_block<1>(v, s, blk);
  if (s == 0 && blk == 0 && t == 0) {
    if (counter) counter[0] = 0;
    if (v.done) v.done[v.nsys] = v.done[v.nsys + 1] = 0;
  }
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  if (blk > 0 && e0 + int64_t(blk) * kThreads >= e1) return;
  const double wn =
      sqrt(sum_partials(npart + first_partial(e0, s, kPartRows),
                        (e1 - e0 + kPartRows - 1) / kPartRows, sh));
  if (blk == 0) reset_state(v, s, wn);
  const int64_t i = e0 + int64_t(blk) * kThreads + t;
  double a = 0.0;
  if (i < e1) {
    const double x = wn > 0.0 ? w[i] / wn : 0.0;
    V[i] = x;
    if (src) {
      const int64_t sp = i / 3;
      src[(i - 3 * sp) * (v.m3 / 3) + sp] = Real(hw[sp] * x);
    }
    if (mw) {
      const double y = wn > 0.0 ? mw[i] / wn : 0.0;
      u[i] = y;
      a = x * y;
    }
  }
  if (!mw) return;
  a = wave_sum(a);
  const int64_t q = int64_t(blk) * (kThreads / 64) + (t >> 6);
  if ((t & 63) == 0 && e0 + q * kPartRows < e1)
    apart[first_partial(e0, s, kPartRows) + q] = a;
}

// Workgroups of a process of `len` elements in lz_dots and lz_update.
template <int EPT>
__device__ __forceinline__ int seg_groups(int64_t len) {
  const int64_t g = (len + kThreads * EPT - 1) / (kThreads * EPT);
  return g > 0 ? int(g) : 1;
}

// Process s's partials of h_j (j < k) and |u|^2 (j = k): one per workgroup, those of j from dots_at + j
// times its workgroups.
template <int EPT>
__device__ __forceinline__ int64_t dots_at(int64_t e0, int s) {
  return (kMaxKrylov + 1) * first_partial(e0, s, kThreads * EPT);
}

template <int EPT>
__global__ __launch_bounds__(kThreads) void lz_dots(SegView v, int k,
                                                    const double *__restrict__ V,
                                                    double *__restrict__ u,
                                                    const double *__restrict__ apart,
                                                    double *__restrict__ part) {
  constexpr int W = kThreads / 64;
  __shared__ double sh[W];
  __shared__ double hsh[(kMaxKrylov + 1) * W];   // wavefront sums: [j * W + wave]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int s, blk;
  seg_block<EPT>(v, s, blk);
  if (v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  const int ng = seg_groups<EPT>(e1 - e0);
  if (blk >= ng) return;
  LzState *st = v.st + s;
  const double *vk = V + int64_t(k - 1) * v.m3;
  const double *vp = V + int64_t(k > 1 ? k - 2 : 0) * v.m3;
  const double be = k > 1 ? st->beta[k - 2] : 0.0;
  bool in[EPT];
  int64_t ix[EPT];
  double x[EPT], xv[EPT], xp[EPT];
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    const int64_t i = e0 + (int64_t(blk) * EPT + r) * kThreads + t;
    in[r] = i < e1;
    ix[r] = in[r] ? i : 0;
    x[r] = in[r] ? u[ix[r]] : 0.0;
    xv[r] = in[r] ? vk[ix[r]] : 0.0;
    xp[r] = in[r] && k > 1 ? vp[ix[r]] : 0.0;
  }
  const double al = sum_partials(apart + first_partial(e0, s, kPartRows),
                                 (e1 - e0 + kPartRows - 1) / kPartRows, sh);
  if (blk == 0 && t == 0) st->alpha[k - 1] = al;
  double nrm = 0.0;
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    x[r] -= al * xv[r];
    x[r] -= be * xp[r];
    if (in[r]) u[ix[r]] = x[r];
    nrm += x[r] * x[r];
  }
  for (int j0 = 0; j0 < k; j0 += 8) {   // eight basis vectors' loads at a time
    double vq[8][EPT], a[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < EPT; ++r) vq[q][r] = V[int64_t(min(j0 + q, k - 1)) * v.m3 + ix[r]];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      a[q] = 0.0;
#pragma unroll
      for (int r = 0; r < EPT; ++r) a[q] += vq[q][r] * x[r];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = wave_sum(a[q]);
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (j0 + q < k) hsh[(j0 + q) * W + wave] = a[q];
  }
  nrm = wave_sum(nrm);
  if (lane == 0) hsh[k * W + wave] = nrm;
  __syncthreads();
  if (t <= k) {
    double r = hsh[t * W];
#pragma unroll
    for (int w = 1; w < W; ++w) r += hsh[t * W + w];
    part[dots_at<EPT>(e0, s) + int64_t(t) * ng + blk] = r;
  }
}

// Where a process reports to the host after iteration k (all nullable): a single process its ring
// slot, the processes of a batch one word each.
struct LzReport {
  LzRingSlot *ring;
  int *words;
  int epoch;
};

__device__ __forceinline__ void report_stop(const SegView &v, int s, int k, bool stop,
                                            const LzReport &rep) {
  if (stop) {
    v.done[s] = 1;
    if (atomicAdd(v.done + v.nsys + 1, 1) + 1 == v.nsys) v.done[v.nsys] = 1;
  }
  // the word says all that the host reads, so it need not wait for earlier stores
  if (rep.words)
    __hip_atomic_store(rep.words + s, lz_tag(rep.epoch, k) | (stop ? kTagStop : 0),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The root of T_k and the stop test of process s by one workgroup, beta_k being in the state.
__device__ __forceinline__ void root_and_stop(const SegView &v, int s, int k, double tol,
                                              const LzReport &rep) {
  LzState *st = v.st + s;
  // every thread reads the same reason: only this workgroup writes it, after the barriers
  if (v.done || st->reason == 0) tridiag_body(k, tol, st, v.eig + s);
  if (threadIdx.x != 0) return;
  if (rep.ring) post_status(st, rep.ring, lz_tag(rep.epoch, k));
  if (v.done) report_stop(v, s, k, st->reason != 0, rep);
}

// The same in a launch of its own, one workgroup per process.
__global__ __launch_bounds__(kThreads) void lz_root(SegView v, int k, double tol, LzReport rep) {
  if (v.done && v.done[blockIdx.x]) return;
  root_and_stop(v, blockIdx.x, k, tol, rep);
}

// ROOT: the process's first workgroup takes the root too.  Its registers and LDS leave two
// workgroups per CU, so a grid beyond that (large batches: 1,536 workgroups took 36 us) leaves
// the root to lz_root.
template <int EPT, typename Real, bool ROOT>
__global__ __launch_bounds__(kThreads, 2) void lz_update(
    SegView v, int k, double tol, double *__restrict__ V, const double *__restrict__ u,
    const double *__restrict__ part, int write_next, const double *__restrict__ hw,
    Real *__restrict__ src, int *counter, LzReport rep) {
  __shared__ double hs[kMaxKrylov + 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int s, blk;
  seg_block<EPT>(v, s, blk);
  if (counter && s == 0 && blk == 0 && t == 0) counter[0] = 0;
  if (v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  const int ng = seg_groups<EPT>(e1 - e0);
  if (blk >= ng) return;
  LzState *st = v.st + s;
  for (int j = wave; j <= k; j += kThreads / 64) {
    const double *p = part + dots_at<EPT>(e0, s) + int64_t(j) * ng;
    double a = 0.0;
    for (int b = lane; b < ng; b += 64) a += p[b];
    a = wave_sum(a);
    if (lane == 0) hs[j] = a;
  }
  __syncthreads();
  const double hj = lane < k ? hs[lane] : 0.0;
  const double b2 = hs[k] - wave_sum(hj * hj);
  const double beta = sqrt(b2 > 0.0 ? b2 : (b2 == b2 ? 0.0 : b2));
  if (write_next) {
    int64_t ix[EPT];
    bool in[EPT];
    double x[EPT], proj[EPT];
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const int64_t i = e0 + (int64_t(blk) * EPT + r) * kThreads + t;
      in[r] = i < e1;
      ix[r] = in[r] ? i : 0;
      x[r] = in[r] ? u[ix[r]] : 0.0;
      proj[r] = 0.0;
    }
    for (int j0 = 0; j0 < k; j0 += 8) {
      double vq[8][EPT];
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int r = 0; r < EPT; ++r) vq[q][r] = V[int64_t(min(j0 + q, k - 1)) * v.m3 + ix[r]];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double h = j0 + q < k ? hs[j0 + q] : 0.0;
#pragma unroll
        for (int r = 0; r < EPT; ++r) proj[r] += h * vq[q][r];
      }
    }
#pragma unroll
    for (int r = 0; r < EPT; ++r)
      if (in[r]) {
        const double y = x[r] - proj[r];
        const double z = beta > 0.0 ? y / beta : 0.0;
        V[int64_t(k) * v.m3 + ix[r]] = z;
        if (src) {
          const int64_t sp = ix[r] / 3;
          src[(ix[r] - 3 * sp) * (v.m3 / 3) + sp] = Real(hw[sp] * z);
        }
      }
  }
  if (blk != 0) return;
  if (t == 0) st->beta[k - 1] = beta;
  if constexpr (ROOT) {
    __syncthreads();
    root_and_stop(v, s, k, tol, rep);
  }
}

// ---- the same iteration with its sums in a fixed grouping (mixed precision) ---------------------
//
// A mixed product rounds v_k to float32, so another rounding of alpha, h or beta, 1e-16 of v_k, now
// and then carries one of its elements across a float32 rounding boundary (a few per cent of the
// solves of 282,000 spheres), which moves a position by 1e-10 and a velocity of the next step by up
// to 7e-8.  Mixed processes therefore keep one grouping of every sum, whatever the launches: NB
// workgroups of strided elements, a tree over the workgroup's threads, then the NB partials by a
// tree (single process, NB = 256) or in order (segments, NB = 16), and beta as the norm of the
// re-orthogonalised u.  Each finishing sum is taken by every workgroup that needs it instead of a
// launch of its own: four kernels per iteration after the product, against six (eight in
// batches, with the packing of v_k and the all-done flag).

template <bool TREE>
constexpr int ord_blocks() { return TREE ? 256 : 16; }

// Sum of the workgroup's 256 values by a tree, on thread 0.
__device__ __forceinline__ double tree_sum(double v, double *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  double r = 0.0;
  if (t < 64) {
    r = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
    r = wave_sum(r);
  }
  __syncthreads();
  return r;
}

// Sum of a quantity's partials, the same on every lane (every lane of a wavefront calls this).
template <bool TREE>
__device__ __forceinline__ double finish_sum(const double *__restrict__ p) {
  if constexpr (TREE) {
    const int l = threadIdx.x & 63;
    return wave_sum((p[l] + p[l + 128]) + (p[l + 64] + p[l + 192]));
  } else {
    double acc = 0.0;
    for (int b = 0; b < ord_blocks<TREE>(); ++b) acc += p[b];
    return acc;
  }
}

// part[s * NB + b]: partial of a . b over process s.
template <bool TREE>
__global__ __launch_bounds__(kThreads) void ord_dot(SegView v, const double *__restrict__ a,
                                                    const double *__restrict__ b, int check_done,
                                                    double *__restrict__ part) {
  __shared__ double sh[kThreads];
  constexpr int NB = ord_blocks<TREE>();
  const int s = blockIdx.y;
  if (check_done && v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  double acc = 0.0;
  for (int64_t i = e0 + int64_t(blockIdx.x) * kThreads + threadIdx.x; i < e1;
       i += int64_t(NB) * kThreads)
    acc += a[i] * b[i];
  const double r = tree_sum(acc, sh);
  if (threadIdx.x == 0) part[int64_t(s) * NB + blockIdx.x] = r;
}

// lz_start from the partials of w . w (alpha_1 is left to ord_dot).
template <bool TREE, typename Real>
__global__ __launch_bounds__(kThreads) void ord_start(SegView v, const double *__restrict__ w,
                                                      const double *__restrict__ npart,
                                                      double *__restrict__ V,
                                                      const double *__restrict__ hw,
                                                      Real *__restrict__ src,
                                                      const double *__restrict__ mw,
                                                      double *__restrict__ u, int *counter) {
  const int t = threadIdx.x;
  int s, blk;
  seg_block<1>(v, s, blk);
  if (s == 0 && blk == 0 && t == 0) {
    if (counter) counter[0] = 0;
    if (v.done) v.done[v.nsys] = v.done[v.nsys + 1] = 0;
  }
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  if (blk > 0 && e0 + int64_t(blk) * kThreads >= e1) return;
  const double wn = sqrt(finish_sum<TREE>(npart + int64_t(s) * ord_blocks<TREE>()));
  if (blk == 0) reset_state(v, s, wn);
  const int64_t i = e0 + int64_t(blk) * kThreads + t;
  if (i >= e1) return;
  const double x = wn > 0.0 ? w[i] / wn : 0.0;
  V[i] = x;
  if (src) {
    const int64_t sp = i / 3;
    src[(i - 3 * sp) * (v.m3 / 3) + sp] = Real(hw[sp] * x);
  }
  if (mw) u[i] = wn > 0.0 ? mw[i] / wn : 0.0;
}

// part[(s * kMaxKrylov + j) * NB + b] = partial of V_j . (u - alpha_k v_k - beta_{k-1} v_{k-1}), j =
// blockIdx.z < k; u is not modified.
template <bool TREE>
__global__ __launch_bounds__(kThreads) void ord_dots(SegView v, int k,
                                                     const double *__restrict__ V,
                                                     const double *__restrict__ u,
                                                     const double *__restrict__ apart,
                                                     double *__restrict__ part) {
  __shared__ double sh[kThreads];
  constexpr int NB = ord_blocks<TREE>();
  const int s = blockIdx.y, j = blockIdx.z;
  if (v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  LzState *st = v.st + s;
  const double al = finish_sum<TREE>(apart + int64_t(s) * NB);
  if (blockIdx.x == 0 && j == 0 && threadIdx.x == 0) st->alpha[k - 1] = al;
  const double *vj = V + int64_t(j) * v.m3, *vk = V + int64_t(k - 1) * v.m3;
  const double *vprev = k > 1 ? V + int64_t(k - 2) * v.m3 : nullptr;
  const double be = vprev ? st->beta[k - 2] : 0.0;
  double acc = 0.0;
  for (int64_t i = e0 + int64_t(blockIdx.x) * kThreads + threadIdx.x; i < e1;
       i += int64_t(NB) * kThreads) {
    double x = u[i] - al * vk[i];
    if (vprev) x -= be * vprev[i];
    acc += vj[i] * x;
  }
  const double r = tree_sum(acc, sh);
  if (threadIdx.x == 0) part[(int64_t(s) * kMaxKrylov + j) * NB + blockIdx.x] = r;
}

// u <- u - alpha_k v_k - beta_{k-1} v_{k-1} - sum_j h_j V_j, and the partials of |u|^2.
template <bool TREE>
__global__ __launch_bounds__(kThreads) void ord_update(SegView v, int k,
                                                       const double *__restrict__ V,
                                                       double *__restrict__ u,
                                                       const double *__restrict__ part,
                                                       double *__restrict__ bpart) {
  __shared__ double sh[kThreads];
  __shared__ double hs[kMaxKrylov];
  constexpr int NB = ord_blocks<TREE>();
  const int s = blockIdx.y, t = threadIdx.x;
  if (v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  LzState *st = v.st + s;
  const double *p = part + int64_t(s) * kMaxKrylov * NB;
  if constexpr (TREE) {
    for (int j = t >> 6; j < k; j += kThreads / 64) {
      const double h = finish_sum<TREE>(p + int64_t(j) * NB);
      if ((t & 63) == 0) hs[j] = h;
    }
  } else {
    if (t < k) hs[t] = finish_sum<TREE>(p + int64_t(t) * NB);
  }
  __syncthreads();
  const double *vk = V + int64_t(k - 1) * v.m3;
  const double *vprev = k > 1 ? V + int64_t(k - 2) * v.m3 : nullptr;
  const double al = st->alpha[k - 1], be = vprev ? st->beta[k - 2] : 0.0;
  double acc = 0.0;
  for (int64_t i = e0 + int64_t(blockIdx.x) * kThreads + t; i < e1;
       i += int64_t(NB) * kThreads) {
    double x = u[i] - al * vk[i];
    if (vprev) x -= be * vprev[i];
    double proj = 0.0;
    for (int j = 0; j < k; ++j) proj += hs[j] * V[int64_t(j) * v.m3 + i];
    x -= proj;
    u[i] = x;
    acc += x * x;
  }
  const double r = tree_sum(acc, sh);
  if (t == 0) bpart[int64_t(s) * NB + blockIdx.x] = r;
}

// beta_k, v_{k+1} = u / beta_k (when write_next) into the basis and the packed sources and, with
// ROOT, the root and stop test by the process's first workgroup (see lz_update).
template <bool TREE, typename Real, bool ROOT>
__global__ __launch_bounds__(kThreads, ROOT ? 2 : 4) void ord_scale(
    SegView v, int k, double tol, double *__restrict__ V, const double *__restrict__ u,
    const double *__restrict__ bpart, int write_next, const double *__restrict__ hw,
    Real *__restrict__ src, int *counter, LzReport rep) {
  const int t = threadIdx.x;
  int s, blk;
  seg_block<1>(v, s, blk);
  if (counter && s == 0 && blk == 0 && t == 0) counter[0] = 0;
  if (v.done && v.done[s]) return;
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  if (blk > 0 && e0 + int64_t(blk) * kThreads >= e1) return;
  const double beta = sqrt(finish_sum<TREE>(bpart + int64_t(s) * ord_blocks<TREE>()));
  const int64_t i = e0 + int64_t(blk) * kThreads + t;
  if (write_next && i < e1) {
    const double x = beta > 0.0 ? u[i] / beta : 0.0;
    V[int64_t(k) * v.m3 + i] = x;
    if (src) {
      const int64_t sp = i / 3;
      src[(i - 3 * sp) * (v.m3 / 3) + sp] = Real(hw[sp] * x);
    }
  }
  if (blk != 0) return;
  if (t == 0) v.st[s].beta[k - 1] = beta;
  if constexpr (ROOT) {
    __syncthreads();
    root_and_stop(v, s, k, tol, rep);
  }
}

// Longest segment (3 n values of one system) that one workgroup takes through a whole Lanczos
// iteration (lanczos_step_body); longer segments use the multi-workgroup reductions.  One
// workgroup keeps too few loads in flight for much longer segments: with 8,192 spheres per
// system the 64-system batched step was 18 % slower than with the separate kernels.
constexpr int64_t kFusedSegment = 3 * 512;

// The vector work and the eigensolve of Lanczos iteration k for the segment [e0, e1) of the
// vectors, by one workgroup, after the product u = M v_k: alpha_k = v_k . u; u -= alpha_k v_k +
// beta_{k-1} v_{k-1}; the full re-orthogonalisation u -= V_k (V_k^T u); beta_k = |u|; the
// eigensolve of T_k with its stop test (tridiag_body); and, unless the process stopped,
// v_{k+1} = u / beta_k (when write_next).  The steps are those of the separate kernels, beta
// as the norm of the re-orthogonalised u (as the ord_ kernels take it, not lz_update); the sums
// are taken over the workgroup instead of in two stages, so that the vector work, root and stop
// test of small systems are one launch per iteration instead of two to five.
// Sums over the workgroup of NV values per thread, each returned to every thread: a butterfly
// over the wavefront's 64 lanes, then the kThreads/64 wavefront sums added in a fixed order.
template <int NV>
__device__ __forceinline__ void group_sums(double (&v)[NV], double *sh) {
  constexpr int W = kThreads / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NV; ++q)
    for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_xor(v[q], off, 64);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < NV; ++q) sh[q * W + wave] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double r = sh[q * W];
    for (int w = 1; w < W; ++w) r += sh[q * W + w];
    v[q] = r;
  }
  __syncthreads();
}

// The vector work (alpha_k, the recurrence, the re-orthogonalisation, beta_k; alpha and beta
// stored in st), leaving the unnormalised u; returns beta_k to every thread.
// The segment has at most kEpt values per thread (kFusedSegment in all), so each thread keeps
// its values of u, v_k and v_{k-1} in registers, and each pass over the basis issues all its
// loads at once; the sums and their order are those of one value at a time.
constexpr int kMaxEpt = int(kFusedSegment / kThreads);
static_assert(kFusedSegment % kThreads == 0, "whole values per thread");
template <int kEpt>
__device__ __forceinline__ double lanczos_vec_values(LzState *__restrict__ st,
                                                     const double *__restrict__ V,
                                                     double *__restrict__ u, int64_t m3,
                                                     int64_t e0, int64_t e1, int k) {
  constexpr int W = kThreads / 64;
  __shared__ double sh[8 * W];
  __shared__ double hsh[kMaxKrylov * W];   // wavefront sums of h_j: [j * W + wave]
  __shared__ double hs[kMaxKrylov];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const double *vk = V + int64_t(k - 1) * m3;
  const double *vp = k > 1 ? V + int64_t(k - 2) * m3 : nullptr;
  // this thread's values: element e0 + t + r kThreads, r < kEpt (clamped loads past e1)
  bool in[kEpt];
  int64_t ix[kEpt];
  double uu[kEpt], xv[kEpt];
#pragma unroll
  for (int r = 0; r < kEpt; ++r) {
    const int64_t i = e0 + t + int64_t(r) * kThreads;
    in[r] = i < e1;
    ix[r] = in[r] ? i : e0;
  }
#pragma unroll
  for (int r = 0; r < kEpt; ++r) uu[r] = u[ix[r]];
#pragma unroll
  for (int r = 0; r < kEpt; ++r) xv[r] = vk[ix[r]];
  double acc[1] = {0.0};
#pragma unroll
  for (int r = 0; r < kEpt; ++r)
    if (in[r]) acc[0] += xv[r] * uu[r];
  group_sums(acc, sh);
  const double alpha = acc[0];
  const double bprev = k > 1 ? st->beta[k - 2] : 0.0;
  double pv[kEpt];
#pragma unroll
  for (int r = 0; r < kEpt; ++r) pv[r] = vp ? vp[ix[r]] : 0.0;
#pragma unroll
  for (int r = 0; r < kEpt; ++r) {
    double x = uu[r] - alpha * xv[r];
    if (vp) x -= bprev * pv[r];
    uu[r] = x;
  }
  // h_j = V_j . u for j < k, eight basis vectors per pass (past the last vector the loads
  // reread it and add nothing); each wavefront's sums go to LDS, added over the wavefronts
  // in a fixed order after the last pass
  for (int j0 = 0; j0 < k; j0 += 8) {
    const int nj = min(8, k - j0);
    double vq[8][kEpt];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < kEpt; ++r) vq[q][r] = V[int64_t(min(j0 + q, k - 1)) * m3 + ix[r]];
    double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < kEpt; ++r)
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (in[r] && q < nj) a[q] += vq[q][r] * uu[r];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      for (int off = 32; off > 0; off >>= 1) a[q] += __shfl_xor(a[q], off, 64);
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < nj) hsh[(j0 + q) * W + wave] = a[q];
  }
  __syncthreads();
  if (t < k) {
    double r = hsh[t * W];
    for (int w = 1; w < W; ++w) r += hsh[t * W + w];
    hs[t] = r;
  }
  __syncthreads();
  // u -= V_k h: per value the terms in increasing j, eight basis vectors' loads at a time
  double proj[kEpt];
#pragma unroll
  for (int r = 0; r < kEpt; ++r) proj[r] = 0.0;
  for (int j0 = 0; j0 < k; j0 += 8) {
    const int nj = min(8, k - j0);
    double vq[8][kEpt];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < kEpt; ++r) vq[q][r] = V[int64_t(min(j0 + q, k - 1)) * m3 + ix[r]];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double hj = q < nj ? hs[j0 + q] : 0.0;
#pragma unroll
      for (int r = 0; r < kEpt; ++r)
        if (q < nj) proj[r] += hj * vq[q][r];
    }
  }
  acc[0] = 0.0;
#pragma unroll
  for (int r = 0; r < kEpt; ++r) {
    uu[r] -= proj[r];
    if (in[r]) {
      u[ix[r]] = uu[r];
      acc[0] += uu[r] * uu[r];
    }
  }
  group_sums(acc, sh);
  const double beta = sqrt(acc[0]);
  if (t == 0) {
    st->alpha[k - 1] = alpha;
    st->beta[k - 1] = beta;
  }
  return beta;
}

// lanczos_vec_values with as many values per thread as the segment needs (workgroup-uniform)
__device__ __forceinline__ double lanczos_vec_body(LzState *__restrict__ st,
                                                   const double *__restrict__ V,
                                                   double *__restrict__ u, int64_t m3,
                                                   int64_t e0, int64_t e1, int k) {
  static_assert(kMaxEpt == 6, "one case per count of values per thread");
  switch (int((e1 - e0 + kThreads - 1) / kThreads)) {
    case 0:
    case 1: return lanczos_vec_values<1>(st, V, u, m3, e0, e1, k);
    case 2: return lanczos_vec_values<2>(st, V, u, m3, e0, e1, k);
    case 3: return lanczos_vec_values<3>(st, V, u, m3, e0, e1, k);
    case 4: return lanczos_vec_values<4>(st, V, u, m3, e0, e1, k);
    case 5: return lanczos_vec_values<5>(st, V, u, m3, e0, e1, k);
    default: return lanczos_vec_values<6>(st, V, u, m3, e0, e1, k);
  }
}

// v_{k+1} = u / beta_k on [e0, e1) (0 when beta_k = 0)
__device__ __forceinline__ void lanczos_write_next(double *__restrict__ V,
                                                   const double *__restrict__ u, int64_t m3,
                                                   int64_t e0, int64_t e1, int k, double beta) {
  double *next = V + int64_t(k) * m3;
  for (int64_t i = e0 + threadIdx.x; i < e1; i += kThreads)
    next[i] = beta > 0.0 ? u[i] / beta : 0.0;
}

// The vector work and the eigensolve of Lanczos iteration k for the segment [e0, e1) of the
// vectors, by one workgroup: lanczos_vec_body, the eigensolve of T_k with its stop test
// (tridiag_body) and, unless the process stopped, v_{k+1} (when write_next).
__device__ void lanczos_step_body(LzState *__restrict__ st, LzEig *__restrict__ eig,
                                  double *__restrict__ V, double *__restrict__ u, int64_t m3,
                                  int64_t e0, int64_t e1, int k, double tol, bool write_next) {
  const double beta = lanczos_vec_body(st, V, u, m3, e0, e1, k);
  __syncthreads();
  tridiag_body(k, tol, st, eig);
  __syncthreads();
  if (write_next && st->reason == 0) lanczos_write_next(V, u, m3, e0, e1, k, beta);
}

// ---- small systems (3 n <= kFusedSegment): one launch per iteration ------------------------------
//
// A few hundred spheres leave every kernel of an iteration at the cost of its launch, so one kernel
// takes the iteration: launch k finishes iteration k - 1 (alpha, the recurrence, the
// re-orthogonalisation, beta, v_k), forms u_k = M v_k, and takes the root and stop test of
// T_{k-2}.  No workgroup waits for another: each one forms v_k for itself (the same sums in
// the same order, from vectors that fit the L2) and then the rows of u_k that it owns, one
// wavefront per row; the last workgroup takes the root, whose coefficients the launches before
// have stored.  All basis vectors' values are loaded at once into registers (twelve wavefronts,
// one or two values per thread), which the projection then reuses.  What bounds an iteration is the
// latency of those loads and of the sums, and the root's chain beside them.  256 spheres, float64:
// 31.6 -> 13.4 us per iteration, 25 of them to 1e-6 870 -> 345 us per solve (four kernels per
// iteration on two streams before, the root's issued by a helper thread).
constexpr int kSmallThreads = 768;

struct SmallArgs {
  LzState *st;
  LzEig *eig;
  double *V;           // basis, max_iter rows
  const double *w;
  const double *mw;    // M w (nullable): u_1 is then M w / |w|
  double *u0, *u1;     // u_k of even and odd k
  int64_t n;
  int k, max_iter;
  int part;            // float32: sources summed in float32 before they are added in float64
  double tol, scale;
  LzReport rep;        // ring: status slot of T_{k-2}
};

// Rows of M F for one target per wavefront.  Float64 sources are dealt to the lanes in turn; float32
// ones in runs of `part` (the runs, and the order within them, of the one-tile product of
// sym_tile_pair, so both give the same float32 sums).
template <bool WALL, bool PERIODIC>
struct SmallRowsD {
  double x[512], y[512], z[512], f[3][512];
  __device__ __forceinline__ void stage(const GeomD &g, int j) {
    x[j] = g.x[j];
    y[j] = g.y[j];
    z[j] = g.z[j];
  }
  __device__ __forceinline__ void row(int n, int, int i, int lane, const PairConsts<double> &k,
                                      double (&acc)[3]) const {
    const double xi = x[i], yi = y[i], zi = z[i];
#pragma unroll 2
    for (int j = lane; j < n; j += 64)
      for_images<PERIODIC>(xi - x[j], yi - y[j], k, [&](double dx, double dy) {
        const double dz = zi - z[j];
        SymCoef<double> c;
        if (dx * dx + dy * dy + dz * dz < kFourA2) {
          sym_coefficients<double, false, false, WALL>(dx, dy, zi, z[j], k, c);
          sym_apply_one<double, WALL>(c, f[0][j], f[1][j], f[2][j], acc[0], acc[1], acc[2]);
        } else {
          sym_coefficients<double, true, false, WALL>(dx, dy, zi, z[j], k, c);
          sym_apply_one<double, WALL>(c, f[0][j], f[1][j], f[2][j], acc[0], acc[1], acc[2]);
        }
      });
  }
};
template <bool WALL, bool PERIODIC>
struct SmallRowsF {
  float xh[512], xl[512], yh[512], yl[512], z[512], f[3][512];
  __device__ __forceinline__ void stage(const GeomF &g, int j) {
    xh[j] = g.xh[j];
    xl[j] = g.xl[j];
    yh[j] = g.yh[j];
    yl[j] = g.yl[j];
    z[j] = g.z[j];
  }
  __device__ __forceinline__ void row(int n, int part, int i, int lane,
                                      const PairConsts<float> &k, double (&acc)[3]) const {
    const float xih = xh[i], xil = xl[i], yih = yh[i], yil = yl[i], zi = z[i];
    for (int j0 = lane * part; j0 < n; j0 += 64 * part) {
      float a[3] = {0.f, 0.f, 0.f};
      const int j1 = min(n, j0 + part);
#pragma unroll 2
      for (int j = j0; j < j1; ++j) {
        const float dx0 = (xih - xh[j]) + (xil - xl[j]);
        const float dy0 = (yih - yh[j]) + (yil - yl[j]);
        for_images<PERIODIC>(dx0, dy0, k, [&](float dx, float dy) {
          const float dz = zi - z[j];
          if (dx * dx + dy * dy + dz * dz < float(kFourA2))
            pair_velocity<float, false, false, WALL>(dx, dy, zi, z[j], f[0][j], f[1][j], f[2][j],
                                                     0.f, 0.f, 0.f, k, a[0], a[1], a[2]);
          else
            pair_velocity<float, false, true, WALL>(dx, dy, zi, z[j], f[0][j], f[1][j], f[2][j],
                                                    0.f, 0.f, 0.f, k, a[0], a[1], a[2]);
        });
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[c] += double(a[c]);
    }
  }
};

template <typename Real, int EPT, bool WALL, bool PERIODIC>
__global__ __launch_bounds__(kSmallThreads) void lz_small(
    SmallArgs A, typename std::conditional<std::is_same<Real, double>::value, GeomD, GeomF>::type g,
    PairConsts<Real> kc) {
  using Rows = typename std::conditional<std::is_same<Real, double>::value,
                                         SmallRowsD<WALL, PERIODIC>,
                                         SmallRowsF<WALL, PERIODIC>>::type;
  constexpr int W = kSmallThreads / 64;
  constexpr int KR = EPT == 1 ? 32 : 16;   // basis vectors kept in registers
  __shared__ Rows R;
  __shared__ double sh[W];
  __shared__ double xs[kSmallThreads * EPT];
  __shared__ double hs[kMaxKrylov + 1];
  __shared__ int stop_s;
  const int k = A.k, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int n = int(A.n), m3 = 3 * n;
  LzState *st = A.st;
  if (blockIdx.x == gridDim.x - 1) {   // the root of T_{k-2}
    if (k < 3 || t >= kThreads) return;
    // every thread reads the same reason: only this workgroup writes it, after the barriers
    if (st->reason == 0) tridiag_body(k - 2, A.tol, st, A.eig);
    if (t == 0) post_status(st, A.rep.ring, lz_tag(A.rep.epoch, k - 2));
    return;
  }
  if (k > A.max_iter + 1) return;   // the last launch takes a root only
  if (k > 1) {   // reason is written by the root's workgroup meanwhile: one thread reads it
    if (t == 0)
      stop_s = __hip_atomic_load(&st->reason, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    __syncthreads();
    if (stop_s) return;
  }
  if (t < n) R.stage(g, t);
  // workgroup sum of one value, the same on every thread
  auto total = [&](double a) {
    a = wave_sum(a);
    if (lane == 0) sh[wave] = a;
    __syncthreads();
    double r = sh[0];
#pragma unroll
    for (int q = 1; q < W; ++q) r += sh[q];
    return r;
  };
  bool in[EPT];
  int ix[EPT];
  double v[EPT];
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    in[r] = t + r * kSmallThreads < m3;
    ix[r] = in[r] ? t + r * kSmallThreads : 0;
  }
  if (k == 1) {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      v[r] = in[r] ? A.w[ix[r]] : 0.0;
      s += v[r] * v[r];
    }
    const double wn = sqrt(total(s));
#pragma unroll
    for (int r = 0; r < EPT; ++r) v[r] = wn > 0.0 ? v[r] / wn : 0.0;
    if (blockIdx.x == 0) {
      reset_state(SegView{nullptr, nullptr, st, nullptr, nullptr, 1, m3, nullptr, nullptr}, 0, wn);
      if (A.mw)
#pragma unroll
        for (int r = 0; r < EPT; ++r)
          if (in[r]) A.u1[ix[r]] = wn > 0.0 ? A.mw[ix[r]] / wn : 0.0;
    }
  } else {
    const int nv = k - 1;   // basis vectors v_1 .. v_{k-1}
    const double *u = (k & 1) ? A.u0 : A.u1;
    const double *vk = A.V + int64_t(nv - 1) * m3;
    const double *vp = A.V + int64_t(nv > 1 ? nv - 2 : 0) * m3;
    const double be = nv > 1 ? st->beta[nv - 2] : 0.0;
    double x[EPT], xv[EPT], xp[EPT], vq[KR][EPT];
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      x[r] = in[r] ? u[ix[r]] : 0.0;
      xv[r] = in[r] ? vk[ix[r]] : 0.0;
      xp[r] = in[r] && nv > 1 ? vp[ix[r]] : 0.0;
    }
    auto load = [&](int j0) {
#pragma unroll
      for (int q = 0; q < KR; ++q)
        if (j0 + q < nv)
#pragma unroll
          for (int r = 0; r < EPT; ++r) vq[q][r] = A.V[int64_t(j0 + q) * m3 + ix[r]];
    };
    load(0);
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < EPT; ++r) s += xv[r] * x[r];
    const double alpha = total(s);
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      x[r] -= alpha * xv[r];
      x[r] -= be * xp[r];
      xs[t + r * kSmallThreads] = x[r];   // zero past the last element
    }
    __syncthreads();
    // one basis vector per wavefront at a time (and |u|^2 as one more), so that a product costs
    // one sum over lanes instead of one in every wavefront
    double xw[W * EPT];
#pragma unroll
    for (int r = 0; r < W * EPT; ++r) xw[r] = xs[lane + 64 * r];
    for (int j = wave; j <= nv; j += W) {
      double a = 0.0;
      if (j < nv) {
        const double *vj = A.V + int64_t(j) * m3;
#pragma unroll
        for (int r = 0; r < W * EPT; ++r) a += vj[min(lane + 64 * r, m3 - 1)] * xw[r];
      } else {
#pragma unroll
        for (int r = 0; r < W * EPT; ++r) a += xw[r] * xw[r];
      }
      a = wave_sum(a);
      if (lane == 0) hs[j] = a;
    }
    __syncthreads();
    // beta^2 = |u|^2 - |h|^2, as in lz_update
    const double hj = lane < nv ? hs[lane] : 0.0;
    const double b2 = hs[nv] - wave_sum(hj * hj);
    const double beta = sqrt(b2 > 0.0 ? b2 : (b2 == b2 ? 0.0 : b2));
    double proj[EPT];
#pragma unroll
    for (int r = 0; r < EPT; ++r) proj[r] = 0.0;
    for (int j0 = 0; j0 < nv; j0 += KR) {
      if (nv > KR) load(j0);
#pragma unroll
      for (int q = 0; q < KR; ++q)
        if (j0 + q < nv) {
          const double h = hs[j0 + q];
#pragma unroll
          for (int r = 0; r < EPT; ++r) proj[r] += h * vq[q][r];
        }
    }
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const double y = x[r] - proj[r];
      v[r] = beta > 0.0 ? y / beta : 0.0;
    }
    if (blockIdx.x == 0) {
      if (t == 0) {
        st->alpha[nv - 1] = alpha;
        st->beta[nv - 1] = beta;
      }
    }
  }
  if (k > A.max_iter) return;
  if (blockIdx.x == 0)
#pragma unroll
    for (int r = 0; r < EPT; ++r)
      if (in[r]) A.V[int64_t(k - 1) * m3 + ix[r]] = v[r];
  if (k == 1 && A.mw) return;   // u_1 is there already
#pragma unroll
  for (int r = 0; r < EPT; ++r)
    if (in[r]) {
      const int sp = ix[r] / 3;
      R.f[ix[r] - 3 * sp][sp] = Real(g.h[sp] * v[r]);
    }
  __syncthreads();
  const int i = int(blockIdx.x) * W + wave;
  if (i >= n) return;
  double acc[3] = {0.0, 0.0, 0.0};
  R.row(n, A.part, i, lane, kc, acc);
#pragma unroll
  for (int c = 0; c < 3; ++c) acc[c] = wave_sum(acc[c]);
  if (lane == 0) {
    double *u = (k & 1) ? A.u1 : A.u0;
#pragma unroll
    for (int c = 0; c < 3; ++c) u[3 * i + c] = A.scale * g.h[i] * acc[c];
  }
}

// The eigensolve of T_1, T_2, ..., T_m in turn (as a Krylov process meets them), row k - 1 of
// ys (m doubles) receiving y_k = |w| T_k^{1/2} e_1 (entries k..m-1 zero); fail[0] = 1 when an
// eigensolve fails.  The stop tests are evaluated but do not stop the sequence.
__global__ __launch_bounds__(kThreads) void tridiag_sequence(int m, LzState *__restrict__ st,
                                                       LzEig *__restrict__ eig,
                                                       double *__restrict__ ys,
                                                       int *__restrict__ fail) {
  const int t = threadIdx.x;
  if (t == 0) fail[0] = 0;
  for (int k = 1; k <= m; ++k) {
    tridiag_body(k, 0.0, st, eig);
    __syncthreads();
    if (t < m) ys[int64_t(k - 1) * m + t] = t < k ? st->y[t] : 0.0;
    if (t == 0 && st->reason == 4) fail[0] = 1;
    __syncthreads();
  }
}

// lanczos_step_body for every live process, one workgroup each (segments <= kFusedSegment); src,
// counter and rep as in lz_update.  Batches, and the single solves that lz_small does not take
// (preconditioned ones, shapes of more than one tile).
template <typename Real>
__global__ __launch_bounds__(kThreads) void seg_lanczos_step(
    SegView v, double *__restrict__ V, double *__restrict__ u, int k, double tol, int write_next,
    const double *__restrict__ hw, Real *__restrict__ src, int *counter, LzReport rep) {
  const int s = blockIdx.x;
  if (counter && s == 0 && threadIdx.x == 0) counter[0] = 0;
  LzState *st = v.st + s;
  if (v.done ? v.done[s] : st->reason) return;   // past its stop nobody reads a status
  int64_t e0, e1;
  seg_range(v, s, e0, e1);
  lanczos_step_body(st, v.eig + s, V, u, v.m3, e0, e1, k, tol, write_next != 0);
  if (src && write_next && st->reason == 0) {
    const double *next = V + int64_t(k) * v.m3;
    for (int64_t i = e0 + threadIdx.x; i < e1; i += kThreads) {   // this thread's own values
      const int64_t sp = i / 3;
      src[(i - 3 * sp) * (v.m3 / 3) + sp] = Real(hw[sp] * next[i]);
    }
  }
  if (threadIdx.x != 0) return;
  if (rep.ring) post_status(st, rep.ring, lz_tag(rep.epoch, k));
  if (v.done) report_stop(v, s, k, st->reason != 0, rep);
}

// out = V_m y_m per system (m = the system's own iteration count)
__global__ void seg_basis_combine(SegView v, int64_t m, const double *__restrict__ V,
                                  double *__restrict__ out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const LzState &st = v.st[v.sys_of[i / 3]];
  double acc = 0.0;
  for (int j = 0; j < st.m; ++j) acc += st.y[j] * V[int64_t(j) * m + i];
  out[i] = acc;
}

// compact status record per system: (m, reason, eps)
__global__ void lz_status_batched(SegView v, int nsys, LzStatus *__restrict__ out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nsys) return;
  out[s].m = v.st[s].m;
  out[s].reason = v.st[s].reason;
  out[s].eps = v.st[s].eps;
}

// y = x / s, or x /= s in place when y == x (square-root preconditioning)
__global__ void divide_by(int64_t m, const double *__restrict__ x, const double *__restrict__ s,
                          double *y) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < m) y[i] = x[i] / s[i];
}

__global__ void multiply_by(int64_t m, double *x, const double *__restrict__ s) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < m) x[i] *= s[i];
}

inline unsigned nblk(int64_t m) { return unsigned((m + kThreads - 1) / kThreads); }


// Grids of the kernels over every process's elements: workgroups of kThreads and of 4 kThreads values.
struct SegGrids {
  BlockList one, four;
};
SegGrids seg_grids(const Batch &b) {
  static_assert(1 << kBlockShift[1] == kThreads && 1 << kBlockShift[2] == 4 * kThreads, "their lists");
  return SegGrids{b.blocks[1], b.blocks[2]};
}
SegGrids one_process_grids(int64_t m3) {
  SegGrids g;
  g.one.total = std::max(1u, nblk(m3));
  g.one.grid.x = unsigned(g.one.total);
  g.four.total = (g.one.total + 3) / 4;
  g.four.grid.x = unsigned(g.four.total);
  return g;
}
inline int64_t launched(const BlockList &b) { return int64_t(b.grid.x) * b.grid.y; }

// Elements per thread of lz_dots and lz_update: one while the grid then fits the device at once (two
// workgroups per CU, by the registers of the root), else four.
inline int ept_of(const SegGrids &g) { return launched(g.one) <= 512 ? 1 : 4; }

// Partial sums of the processes' scalars: float64 processes take one partial of |w|^2 and of
// alpha per 64 rows and one of each basis product per workgroup of lz_dots, mixed ones the
// grouping of the ord_ kernels.
struct LzPartials {
  double *norm, *alpha, *dots;   // dots: basis products, then |u|^2
};
inline bool one_process(const SegView &v) { return v.offs == nullptr; }

// vectors: the separate kernels of an iteration run (no fused workgroup per process).
int lz_partials(rpb_ctx *ctx, const SegView &v, const SegGrids &g, bool f64, bool vectors,
                LzPartials *out) {
  const int64_t ns = v.nsys;
  const int64_t nb = one_process(v) ? ord_blocks<true>() : ord_blocks<false>();
  const int64_t scalar = f64 ? first_partial(v.m3, ns, kPartRows) + 1 : ns * nb;
  const int64_t groups = f64 ? first_partial(v.m3, ns, kThreads * ept_of(g)) + 1 : ns * nb;
  const int64_t dots = vectors ? (kMaxKrylov + 1) * groups : 0;
  int st;
  out->norm = static_cast<double *>(
      workspace(ctx, WS_REDUCE, size_t(2 * scalar + dots) * sizeof(double), &st));
  if (!out->norm) return st;
  out->alpha = out->norm + scalar;
  out->dots = out->alpha + scalar;
  return RPB_OK;
}

// Whether every process's sums keep the grouping of the ord_ kernels.
template <typename Real>
constexpr bool ordered_sums() { return std::is_same<Real, float>::value; }

// |w|, v_1 and the state of every process.
template <typename Real>
int start_processes(rpb_ctx *ctx, const SegView &v, const SegGrids &g, const double *w,
                    const LzPartials &P, double *V, const double *hw, Real *src, const double *mw,
                    double *u, int *counter, hipStream_t stream) {
  const dim3 grid = g.one.grid;
  if constexpr (ordered_sums<Real>()) {
    auto run = [&](auto T) -> int {
      constexpr bool kT = decltype(T)::value;
      const dim3 dg{unsigned(ord_blocks<kT>()), unsigned(v.nsys), 1u};
      ord_dot<kT><<<dg, kThreads, 0, stream>>>(v, w, w, 0, P.norm);
      RPB_LAUNCHED(ctx);
      ord_start<kT, Real><<<grid, kThreads, 0, stream>>>(v, w, P.norm, V, hw, src, mw, u, counter);
      RPB_LAUNCHED(ctx);
      return RPB_OK;
    };
    return one_process(v) ? run(std::true_type{}) : run(std::false_type{});
  } else {
    lz_dot<<<grid, kThreads, 0, stream>>>(v, w, w, 0, P.norm);
    RPB_LAUNCHED(ctx);
    lz_start<Real><<<grid, kThreads, 0, stream>>>(v, w, P.norm, V, hw, src, mw, u, P.alpha,
                                                  counter);
    RPB_LAUNCHED(ctx);
    return RPB_OK;
  }
}

// The vector work, root and stop test of iteration k of every process after u = M v_k; dotted:
// alpha's partials are there already.
template <typename Real>
int iterate_processes(rpb_ctx *ctx, const SegView &v, const SegGrids &g, int k, double tol,
                      double *V, double *u, bool dotted, const LzPartials &P, bool write_next,
                      const double *hw, Real *src, int *counter, const LzReport &rep,
                      hipStream_t stream) {
  const double *vk = V + int64_t(k - 1) * v.m3;
  const unsigned ns = unsigned(v.nsys);
  const dim3 all = g.one.grid;
  auto root = [&]() -> int {
    lz_root<<<ns, kThreads, 0, stream>>>(v, k, tol, rep);
    RPB_LAUNCHED(ctx);
    return RPB_OK;
  };
  if constexpr (ordered_sums<Real>()) {
    auto run = [&](auto T) -> int {
      constexpr bool kT = decltype(T)::value;
      constexpr unsigned NB = unsigned(ord_blocks<kT>());
      double *bpart = P.dots + int64_t(v.nsys) * kMaxKrylov * NB;
      ord_dot<kT><<<dim3{NB, ns, 1u}, kThreads, 0, stream>>>(v, vk, u, 1, P.alpha);
      RPB_LAUNCHED(ctx);
      ord_dots<kT><<<dim3{NB, ns, unsigned(k)}, kThreads, 0, stream>>>(v, k, V, u, P.alpha,
                                                                       P.dots);
      RPB_LAUNCHED(ctx);
      ord_update<kT><<<dim3{NB, ns, 1u}, kThreads, 0, stream>>>(v, k, V, u, P.dots, bpart);
      RPB_LAUNCHED(ctx);
      if (launched(g.one) <= 512) {
        ord_scale<kT, Real, true><<<all, kThreads, 0, stream>>>(
            v, k, tol, V, u, bpart, write_next, hw, src, counter, rep);
        RPB_LAUNCHED(ctx);
        return RPB_OK;
      }
      ord_scale<kT, Real, false><<<all, kThreads, 0, stream>>>(
          v, k, tol, V, u, bpart, write_next, hw, src, counter, rep);
      RPB_LAUNCHED(ctx);
      return root();
    };
    return one_process(v) ? run(std::true_type{}) : run(std::false_type{});
  } else {
    if (!dotted) {
      lz_dot<<<all, kThreads, 0, stream>>>(v, vk, u, 1, P.alpha);
      RPB_LAUNCHED(ctx);
    }
    const int ept = ept_of(g);
    auto run = [&](auto E, auto R) -> int {
      constexpr int kE = decltype(E)::value;
      constexpr bool kR = decltype(R)::value;
      const dim3 grid = kE == 1 ? g.one.grid : g.four.grid;
      lz_dots<kE><<<grid, kThreads, 0, stream>>>(v, k, V, u, P.alpha, P.dots);
      RPB_LAUNCHED(ctx);
      lz_update<kE, Real, kR><<<grid, kThreads, 0, stream>>>(v, k, tol, V, u, P.dots, write_next,
                                                             hw, src, counter, rep);
      RPB_LAUNCHED(ctx);
      return kR ? RPB_OK : root();
    };
    using E1 = std::integral_constant<int, 1>;
    using E4 = std::integral_constant<int, 4>;
    if (ept == 1) return run(E1{}, std::true_type{});
    if (launched(g.four) <= 512) return run(E4{}, std::true_type{});
    return run(E4{}, std::false_type{});
  }
}

}  // namespace

namespace {

// Outcome of a single-system solve, as the host read it.
struct LzOutcome {
  int m = 0;           // iterations whose result counts
  int reason = 0;
  double eps = 0.0;
};

// Reads the statuses of the iterations up to qmax, in order, until one reports a stop.
int read_statuses(rpb_ctx *ctx, int epoch, int qmax, int *next_q, LzOutcome *out,
                  hipStream_t stream) {
  LzRing *ring = lz_ring(ctx);
  for (; *next_q <= qmax && out->reason == 0; ++*next_q) {
    const int q = *next_q;
    LzRingSlot &slot = ring->slot[q % kLzRing];
    RPB_TRY(wait_pinned(ctx, stream, [&] {
      return __atomic_load_n(&slot.tag, __ATOMIC_ACQUIRE) == lz_tag(epoch, q);
    }));
    out->m = q;
    out->reason = slot.reason;
    out->eps = slot.eps;
  }
  return RPB_OK;
}

// The small-system solve (lz_small).  The status of T_m comes from launch m + 2, and the host reads
// it once launch m + 3 is enqueued, so the device always has one launch queued; launches past
// the stop return at once.
template <typename Real, typename Geom>
int small_solve(rpb_ctx *ctx, const rpb_params *p, const Geom &geom, int part, SmallArgs A,
                LzOutcome *out, hipStream_t stream) {
  constexpr int W = kSmallThreads / 64;
  const unsigned grid = unsigned((A.n + W - 1) / W) + 1u;
  const auto kc = make_pair_consts<Real>(p->lx / p->a, p->ly / p->a);
  A.part = part;
  auto launch = [&](auto E) {
    constexpr int kE = decltype(E)::value;
    auto by_wall = [&](auto Wl) {
      constexpr bool kW = decltype(Wl)::value;
      if (p->lx > 0.0)
        lz_small<Real, kE, kW, true><<<grid, kSmallThreads, 0, stream>>>(A, geom, kc);
      else
        lz_small<Real, kE, kW, false><<<grid, kSmallThreads, 0, stream>>>(A, geom, kc);
    };
    if (p->wall)
      by_wall(std::true_type{});
    else
      by_wall(std::false_type{});
  };
  LzRing *ring_dev = lz_ring_dev(ctx);
  int next_q = 1;
  size_t mark[kLzRing] = {};
  for (int k = 1; k <= A.max_iter + 2 && out->reason == 0; ++k) {
    A.k = k;
    const int m = k - 2;   // the status that this launch writes
    A.rep.ring = m > 0 ? &ring_dev->slot[m % kLzRing] : nullptr;
    mark[k % kLzRing] = ctx->ev_start.size();
    const bool product = k <= A.max_iter && !(k == 1 && A.mw);
    hipEvent_t t0 = nullptr;
    if (product) RPB_TRY(timing_begin(ctx, stream, &t0));
    if (3 * A.n <= kSmallThreads)
      launch(std::integral_constant<int, 1>{});
    else
      launch(std::integral_constant<int, 2>{});
    RPB_LAUNCHED(ctx);
    if (product)
      RPB_TRY(timing_end(ctx, stream, t0, double(A.n) * double(A.n),
                         std::is_same<Real, double>::value ? 0 : 2));
    if (m < 1) continue;
    const int before = next_q;
    RPB_TRY(read_statuses(ctx, A.rep.epoch, k < A.max_iter + 2 ? m - 1 : m, &next_q, out, stream));
    // products past the stop count for nothing
    if (out->reason != 0 && next_q > before && out->m + 1 <= k)
      timing_discard(ctx, mark[(out->m + 1) % kLzRing]);
  }
  return RPB_OK;
}

}  // namespace

int lanczos_run(rpb_ctx *ctx, const rpb_params *p, const Packed &g, const double *w, double tol,
                int max_iter, bool precond, double *out, int *iters, double *eps_out,
                hipStream_t stream, const double *mw) {
  const int64_t n = g.n;
  const int64_t m3 = 3 * n;
  int st;
  double *L = nullptr, *t = nullptr;
  if (precond) {
    L = static_cast<double *>(workspace(ctx, WS_PRECOND, size_t(2 * m3) * sizeof(double), &st));
    if (!L) return st;
    t = L + m3;
    RPB_TRY(block_diag_scale(ctx, p, g, L, stream));
  }
  double *V = static_cast<double *>(
      workspace(ctx, WS_KRYLOV, size_t(max_iter) * size_t(m3) * sizeof(double), &st));
  if (!V) return st;
  double *u = static_cast<double *>(workspace(ctx, WS_VEC_A, size_t(m3) * sizeof(double), &st));
  if (!u) return st;
  LzState *ls = static_cast<LzState *>(workspace(ctx, WS_SMALL, kSmallBytes, &st));
  if (!ls) return st;
  LzEig *eig = static_cast<LzEig *>(workspace(ctx, WS_LZEIG, sizeof(LzEig), &st));
  if (!eig) return st;
  const int epoch = next_epoch(ctx);
  const bool f64 = g.precision == RPB_FP64;
  LzOutcome o;
  const int part = precond || m3 > kFusedSegment ? 0 : one_tile_part(ctx, g);
  if (part > 0) {   // one launch per iteration
    double *u2 = static_cast<double *>(workspace(ctx, WS_LZ_U2, size_t(m3) * sizeof(double), &st));
    if (!u2) return st;
    const SmallArgs A{ls,   eig, V, w, mw, u, u2, n, 1, max_iter, part,
                      tol, 1.0 / (8.0 * M_PI * p->eta * p->a), LzReport{nullptr, nullptr, epoch}};
    if (f64)
      RPB_TRY((small_solve<double>(ctx, p, geom_d(g), part, A, &o, stream)));
    else
      RPB_TRY((small_solve<float>(ctx, p, geom_f(g), part, A, &o, stream)));
  } else {
    // without the preconditioner the kernels that form v_1 and v_{k+1} also pack them for the
    // next product
    const bool prepack = !precond;
    void *src = nullptr;
    if (prepack) {
      src = source_buffer(ctx, g, &st);
      if (!src) return st;
    }
    const double *hw = prepack ? packed_weights(g) : nullptr;
    const SegView view{nullptr, nullptr, ls, nullptr, eig, 1, m3, nullptr, nullptr};
    const SegGrids grids = one_process_grids(m3);
    LzPartials P;
    // Small systems: one launch of one workgroup for the vector work, root and stop test instead of
    // three (float64) or four (mixed).  40 preconditioned iterations, us, separate / one: mixed 64
    // spheres 1,925 / 1,590, 512: 1,985 / 2,005 (20 iterations 900 / 860); float64 64: 1,635 / 1,460,
    // 256: 1,750 / 1,665, 512: 1,810 / 1,925.
    const bool fused = m3 <= (f64 ? kFusedSegment / 2 : kFusedSegment);
    RPB_TRY(lz_partials(ctx, view, grids, f64, !fused, &P));
    if (f64)
      RPB_TRY(start_processes(ctx, view, grids, w, P, V, hw, static_cast<double *>(src), mw, u,
                              nullptr, stream));
    else
      RPB_TRY(start_processes(ctx, view, grids, w, P, V, hw, static_cast<float *>(src), mw, u,
                              nullptr, stream));
    LzRing *ring_dev = lz_ring_dev(ctx);
    const int *stopped = &ls->reason;
    size_t mark[kLzRing] = {};   // first timing record of each iteration in flight
    int next_q = 1;              // first iteration whose status the host has not read
    // The host reads the status of iteration m only after iteration m + 1 has been enqueued, so
    // the device never idles while the host decides.  An iteration past the stop leaves the
    // result unchanged: its product returns at once, and its vector work touches only u, V's
    // next column, the packed sources and entries of alpha and beta past the last iteration.
    for (int k = 1; k <= max_iter && o.reason == 0; ++k) {
      const int slot = k % kLzRing;
      mark[slot] = ctx->ev_start.size();
      double *vm = V + int64_t(k - 1) * m3;
      bool dotted = false;   // alpha's partials are in P
      if (precond) {   // u = L^-1 M L^-1 vm
        divide_by<<<nblk(m3), kThreads, 0, stream>>>(m3, vm, L, t);
        RPB_LAUNCHED(ctx);
        RPB_TRY(matvec_packed(ctx, p, g, t, nullptr, 0, n, u, stream, stopped));
        divide_by<<<nblk(m3), kThreads, 0, stream>>>(m3, u, L, u);
        RPB_LAUNCHED(ctx);
      } else if (k == 1 && mw) {   // M v_1 = (M w) / |w| from the caller's product (lz_start)
        dotted = true;
      } else {   // v_k packed where it was formed
        DotOut dot{f64 && !fused ? vm : nullptr, P.alpha};
        RPB_TRY(matvec_prepacked(ctx, p, g, src, u, stream, stopped, &dot));
        dotted = dot.done;
      }
      const LzReport rep{&ring_dev->slot[slot], nullptr, epoch};
      if (fused) {
        if (f64)
          seg_lanczos_step<double><<<1, kThreads, 0, stream>>>(
              view, V, u, k, tol, k < max_iter, hw, static_cast<double *>(src), nullptr, rep);
        else
          seg_lanczos_step<float><<<1, kThreads, 0, stream>>>(
              view, V, u, k, tol, k < max_iter, hw, static_cast<float *>(src), nullptr, rep);
        RPB_LAUNCHED(ctx);
      } else if (f64)
        RPB_TRY(iterate_processes(ctx, view, grids, k, tol, V, u, dotted, P, k < max_iter, hw,
                                  static_cast<double *>(src), nullptr, rep, stream));
      else
        RPB_TRY(iterate_processes(ctx, view, grids, k, tol, V, u, dotted, P, k < max_iter, hw,
                                  static_cast<float *>(src), nullptr, rep, stream));
      RPB_TRY(read_statuses(ctx, epoch, k < max_iter ? k - 1 : k, &next_q, &o, stream));
      // launches past the stop returned at once: drop their timing records
      if (o.reason != 0 && o.m < k) timing_discard(ctx, mark[(o.m + 1) % kLzRing]);
    }
  }
  const int m = o.m, reason = o.reason;
  const double eps = o.eps;
  basis_combine<<<nblk(m3), kThreads, 0, stream>>>(m3, m, V, ls->y, out);
  RPB_LAUNCHED(ctx);
  if (precond) {
    multiply_by<<<nblk(m3), kThreads, 0, stream>>>(m3, out, L);
    RPB_LAUNCHED(ctx);
  }
  if (iters) *iters = m;
  if (eps_out) *eps_out = eps;
  if (reason == 4) return fail(ctx, RPB_EDEVICE, "tridiagonal eigensolve did not converge");
  if (reason == 3) return fail(ctx, RPB_ENOTSPD, "negative Ritz value at m = %d", m);
  if (reason == 0)
    return fail(ctx, RPB_ENOCONV, "Lanczos: eps = %.3e > tol = %.3e after %d iterations", eps,
                tol, m);
  return RPB_OK;
}


namespace {

// Layout of the batched state: LzState records, the flags of SegView::done, then the status.
inline size_t lz_status_offset(int nsys) {
  return (size_t(nsys) * sizeof(LzState) + size_t(nsys + 2) * sizeof(int) + 255) / 256 * 256;
}

// A product of lanczos_segments: u = M v_k for every process not yet done.
struct SegProduct {
  const double *vk;        // the basis vectors ([3 n] of all processes)
  const void *src;         // v_k packed (NULL: not packed)
  const int *done_dev;     // device flags
  const int *done_host;    // the flags as of the last host read, NULL when unknown
  DotOut dot;              // alpha's partials, when the product can take them
};

// One Krylov process per segment (system) of `b`; product(SegProduct &, u) writes u = M v_k for
// every segment not yet done.  hw (nullable): weights with which v_k is packed for the product where
// it is formed (into `src`, of the precision `f64` names); counter (nullable): the product's work
// counter, zeroed with it.  L (nullable): preconditioner scale, 3 b.n entries, with scratch t.
// mw (nullable, not with L): M w computed by the caller, used for the first iteration.  With
// sync_each the host reads the flags of iteration k after it has enqueued iteration k + lag.
template <typename Product>
int lanczos_segments(rpb_ctx *ctx, const Batch &b, const double *L, double *t, const double *w,
                     double tol, int max_iter, Product &&product, const double *hw, void *src,
                     bool f64, int *counter, double *out, bool sync_each, int lag,
                     LzStatus *status_host, hipStream_t stream, const double *mw = nullptr) {
  const int64_t m3 = 3 * b.n;
  const int nsys = b.nsys;
  bool fused = true;            // every system small enough for one workgroup per iteration
  for (int s = 0; s < nsys; ++s) {
    const int64_t len = 3 * (b.host_offs[s + 1] - b.host_offs[s]);
    fused = fused && len <= kFusedSegment;
  }
  int st;
  double *V = static_cast<double *>(
      workspace(ctx, WS_KRYLOV, size_t(max_iter) * size_t(m3) * sizeof(double), &st));
  if (!V) return st;
  double *u = static_cast<double *>(workspace(ctx, WS_VEC_A, size_t(m3) * sizeof(double), &st));
  if (!u) return st;
  const SegGrids grids = seg_grids(b);
  const size_t states_bytes = size_t(nsys) * sizeof(LzState);
  const size_t status_off = lz_status_offset(nsys);
  char *lz = static_cast<char *>(
      workspace(ctx, WS_LZBATCH, status_off + size_t(nsys) * sizeof(LzStatus), &st));
  if (!lz) return st;
  LzEig *eig = static_cast<LzEig *>(workspace(ctx, WS_LZEIG, size_t(nsys) * sizeof(LzEig), &st));
  if (!eig) return st;
  const SegView v{b.offs, b.sys_of, reinterpret_cast<LzState *>(lz),
                  reinterpret_cast<int *>(lz + states_bytes), eig, nsys, m3,
                  grids.one.list, grids.four.list};
  LzPartials P;
  RPB_TRY(lz_partials(ctx, v, grids, f64, !fused, &P));
  LzStatus *status_dev = reinterpret_cast<LzStatus *>(lz + status_off);
  const unsigned ns = unsigned(nsys);
  // every process reports each iteration into its word of the pinned buffer
  LzReport rep{nullptr, nullptr, next_epoch(ctx)};
  int *words = nullptr;
  if (sync_each) {
    words = reinterpret_cast<int *>(static_cast<char *>(host_scratch(ctx)) + kHostDoneOffset);
    rep.words =
        reinterpret_cast<int *>(static_cast<char *>(host_scratch_dev(ctx)) + kHostDoneOffset);
  }
  std::vector<int> known;   // host copy of the flags, once read

  if (f64)
    RPB_TRY(start_processes(ctx, v, grids, w, P, V, hw, static_cast<double *>(src), mw, u,
                            counter, stream));
  else
    RPB_TRY(start_processes(ctx, v, grids, w, P, V, hw, static_cast<float *>(src), mw, u, counter,
                            stream));
  size_t mark[kLzRing] = {};   // first timing record of each iteration in flight
  int next_q = 1;              // first iteration whose flags the host has not read
  bool stop = false;
  for (int k = 1; k <= max_iter && !stop; ++k) {
    const int slot = k % kLzRing;
    mark[slot] = ctx->ev_start.size();
    double *vk = V + int64_t(k - 1) * m3;
    SegProduct job{vk, src, v.done, known.empty() ? nullptr : known.data(),
                   DotOut{fused || !f64 ? nullptr : vk, P.alpha}};
    if (L) {   // u = L^-1 M L^-1 vk (rows of finished systems are not used)
      divide_by<<<nblk(m3), kThreads, 0, stream>>>(m3, vk, L, t);
      RPB_LAUNCHED(ctx);
      job.vk = t;
      job.dot.v = nullptr;
      RPB_TRY(product(job, u));
      divide_by<<<nblk(m3), kThreads, 0, stream>>>(m3, u, L, u);
      RPB_LAUNCHED(ctx);
    } else if (k == 1 && mw) {   // M v_1 = (M w) / |w| per system (lz_start)
      job.dot.done = true;
    } else {
      RPB_TRY(product(job, u));
    }
    const bool next = k < max_iter;
    if (fused) {   // every system's iteration in one workgroup
      if (f64)
        seg_lanczos_step<double><<<ns, kThreads, 0, stream>>>(
            v, V, u, k, tol, next, hw, static_cast<double *>(src), counter, rep);
      else
        seg_lanczos_step<float><<<ns, kThreads, 0, stream>>>(
            v, V, u, k, tol, next, hw, static_cast<float *>(src), counter, rep);
      RPB_LAUNCHED(ctx);
    } else {
      if (f64)
        RPB_TRY(iterate_processes(ctx, v, grids, k, tol, V, u, job.dot.done, P, next, hw,
                                  static_cast<double *>(src), counter, rep, stream));
      else
        RPB_TRY(iterate_processes(ctx, v, grids, k, tol, V, u, job.dot.done, P, next, hw,
                                  static_cast<float *>(src), counter, rep, stream));
    }
    if (!sync_each) continue;
    const int qmax = next ? k - lag : next_q - 1;   // nothing to decide after the last iteration
    for (; next_q <= qmax && !stop; ++next_q) {
      known.resize(size_t(nsys));
      bool all = true;
      for (int s = 0; s < nsys; ++s) {
        // a stopped process keeps its last word; the others count up
        int word = 0;
        RPB_TRY(wait_pinned(ctx, stream, [&] {
          word = __atomic_load_n(words + s, __ATOMIC_ACQUIRE);
          return (word >> 8) == rep.epoch &&
                 ((word & kTagStop) != 0 || (word & (kTagStop - 1)) >= next_q);
        }));
        known[size_t(s)] = (word & kTagStop) != 0 && (word & (kTagStop - 1)) <= next_q;
        all = all && known[size_t(s)];
      }
      if (all) {
        // launches past the stop returned at once: drop their timing records
        if (next_q < k) timing_discard(ctx, mark[(next_q + 1) % kLzRing]);
        stop = true;
      }
    }
  }
  seg_basis_combine<<<nblk(m3), kThreads, 0, stream>>>(v, m3, V, out);
  RPB_LAUNCHED(ctx);
  if (L) {
    multiply_by<<<nblk(m3), kThreads, 0, stream>>>(m3, out, L);
    RPB_LAUNCHED(ctx);
  }
  lz_status_batched<<<(ns + 63) / 64, 64, 0, stream>>>(v, nsys, status_dev);
  RPB_LAUNCHED(ctx);
  if (status_host) {
    RPB_HIP(ctx, hipMemcpyAsync(status_host, status_dev, size_t(nsys) * sizeof(LzStatus),
                                hipMemcpyDeviceToHost, stream));
    RPB_HIP(ctx, hipStreamSynchronize(stream));
  }
  return RPB_OK;
}

}  // namespace

int lanczos_batched_run(rpb_ctx *ctx, const rpb_params *p, const Batch &b, const Packed &g,
                        const double *w, double tol, int max_iter, bool precond, double *out,
                        bool sync_each, LzStatus *status_host, hipStream_t stream,
                        const double *mw) {
  const int64_t m3 = 3 * b.n;
  int st;
  double *L = nullptr, *t = nullptr;
  if (precond) {
    L = static_cast<double *>(workspace(ctx, WS_PRECOND, size_t(2 * m3) * sizeof(double), &st));
    if (!L) return st;
    t = L + m3;
    RPB_TRY(block_diag_scale(ctx, p, g, L, stream));
  }
  const bool f64 = g.precision == RPB_FP64;
  void *src = nullptr;
  int *counter = nullptr;
  if (!precond) {
    src = source_buffer(ctx, g, &st);
    if (!src) return st;
    counter = work_counter(ctx, &st);
    if (!counter) return st;
  }
  auto product = [&](SegProduct &job, double *u) {
    if (!precond)
      return matvec_batched_prepacked(ctx, p, b, g, job.src, job.done_dev, u, stream, &job.dot);
    return matvec_batched(ctx, p, b, g, job.vk, nullptr, job.done_dev, u, stream);
  };
  return lanczos_segments(ctx, b, L, t, w, tol, max_iter, product,
                          precond ? nullptr : packed_weights(g), src, f64, counter, out, sync_each,
                          1, status_host, stream, precond ? nullptr : mw);
}

int lanczos_batched_status_copy(rpb_ctx *ctx, int nsys, LzStatus *host, hipStream_t stream) {
  const size_t status_off = lz_status_offset(nsys);
  const DevBuf &b = ctx->ws[WS_LZBATCH];
  if (!b.ptr || b.bytes < status_off + size_t(nsys) * sizeof(LzStatus))
    return fail(ctx, RPB_EINVAL, "no batched Lanczos state");
  RPB_HIP(ctx, hipMemcpyAsync(host, static_cast<char *>(b.ptr) + status_off,
                              size_t(nsys) * sizeof(LzStatus), hipMemcpyDeviceToHost, stream));
  RPB_HIP(ctx, hipStreamSynchronize(stream));
  return RPB_OK;
}

int lanczos_status_code(rpb_ctx *ctx, const LzStatus *s, int nsys) {
  int worst = RPB_OK;
  for (int q = 0; q < nsys; ++q) {
    if (s[q].reason == 4)
      return fail(ctx, RPB_EDEVICE, "tridiagonal eigensolve failed (system %d)", q);
    if (s[q].reason == 3) worst = fail(ctx, RPB_ENOTSPD, "negative Ritz value (system %d)", q);
    if (s[q].reason == 0 && worst == RPB_OK)
      worst = fail(ctx, RPB_ENOCONV, "Lanczos tolerance not met (system %d, eps %.3e)", q,
                   s[q].eps);
  }
  return worst;
}

}  // namespace rpb

using namespace rpb;

namespace {

int lanczos_entry(rpb_ctx *ctx, const rpb_params *p, int64_t n, const double *pos,
                  const double *w, double tol, int max_iter, bool precond, double *out,
                  int *iters_out, double *eps_out, rpb_stream_t stream_) {
  RPB_TRY(check_params(ctx, p));
  if (n < 0) return fail(ctx, RPB_EINVAL, "n must be >= 0");
  if (!(tol > 0.0)) return fail(ctx, RPB_EINVAL, "tol must be > 0");
  if (max_iter < 1 || max_iter > kMaxKrylov)
    return fail(ctx, RPB_EINVAL, "max_iter must be in [1, %d]", kMaxKrylov);
  if (iters_out) *iters_out = 0;
  if (eps_out) *eps_out = 0.0;
  if (n == 0) return RPB_OK;
  if (!pos || !w || !out) return fail(ctx, RPB_EINVAL, "pos, w and out must not be NULL");
  const size_t nb = size_t(n) * 3 * sizeof(double);
  if (overlaps(out, nb, pos, nb) || overlaps(out, nb, w, nb))
    return fail(ctx, RPB_EINVAL, "out overlaps an input");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  RPB_HIP(ctx, hipSetDevice(ctx->device));
  Check check;
  RPB_TRY(check_begin(ctx, &check, stream));
  Packed g;
  RPB_TRY(pack_checked(ctx, p, n, pos, WS_GEOM, &g, check, nullptr, Torque{}, nullptr, stream));
  RPB_TRY(check_end(ctx, check, stream));
  const int lz =
      lanczos_run(ctx, p, g, w, tol, max_iter, precond, out, iters_out, eps_out, stream);
  if (lz != RPB_OK && lz != RPB_ENOCONV) return lz;
  RPB_TRY(check_output(ctx, out, 3 * n, stream, "the Brownian increment"));
  return lz;
}

}  // namespace

extern "C" int lanczos_sqrt_apply(rpb_ctx *ctx, const rpb_params *p, int64_t n, const double *pos,
                                  const double *w, double tol, int max_iter, double *out,
                                  int *iters_out, double *eps_out, rpb_stream_t stream) {
  return lanczos_entry(ctx, p, n, pos, w, tol, max_iter, false, out, iters_out, eps_out, stream);
}

extern "C" int lanczos_sqrt_apply_precond(rpb_ctx *ctx, const rpb_params *p, int64_t n,
                                          const double *pos, const double *w, double tol,
                                          int max_iter, double *out, int *iters_out,
                                          double *eps_out, rpb_stream_t stream) {
  return lanczos_entry(ctx, p, n, pos, w, tol, max_iter, true, out, iters_out, eps_out, stream);
}

extern "C" int lanczos_sqrt_apply_batched(rpb_ctx *ctx, const rpb_params *p, int32_t nsys,
                                          const int64_t *offs, const double *pos,
                                          const double *w, double tol, int max_iter, double *out,
                                          int *iters_out, double *eps_out, rpb_stream_t stream_) {
  RPB_TRY(check_params(ctx, p));
  RPB_TRY(check_offsets(ctx, nsys, offs));
  if (p->lx > 0.0)
    return fail(ctx, RPB_EINVAL, "pseudo-periodic boundaries are supported for single systems");
  if (nsys > kMaxBatchSystems)
    return fail(ctx, RPB_EINVAL, "at most %d systems per batch", kMaxBatchSystems);
  if (!(tol > 0.0)) return fail(ctx, RPB_EINVAL, "tol must be > 0");
  if (max_iter < 1 || max_iter > kMaxKrylov)
    return fail(ctx, RPB_EINVAL, "max_iter must be in [1, %d]", kMaxKrylov);
  const int64_t n = offs[nsys];
  for (int s = 0; s < nsys; ++s) {
    if (iters_out) iters_out[s] = 0;
    if (eps_out) eps_out[s] = 0.0;
  }
  if (n == 0) return RPB_OK;
  if (!pos || !w || !out) return fail(ctx, RPB_EINVAL, "pos, w and out must not be NULL");
  const size_t nb = size_t(n) * 3 * sizeof(double);
  if (overlaps(out, nb, pos, nb) || overlaps(out, nb, w, nb))
    return fail(ctx, RPB_EINVAL, "out overlaps an input");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  RPB_HIP(ctx, hipSetDevice(ctx->device));
  RPB_TRY(check_finite(ctx, pos, n, stream));
  Batch b;
  RPB_TRY(prepare_batch(ctx, nsys, offs, p->precision, &b, stream));
  Packed g;
  RPB_TRY(pack_geometry(ctx, p, n, pos, WS_GEOM, &g, stream));
  LzStatus *stat = static_cast<LzStatus *>(host_scratch(ctx));
  RPB_TRY(lanczos_batched_run(ctx, p, b, g, w, tol, max_iter, false, out, true, stat, stream));
  for (int s = 0; s < nsys; ++s) {
    if (iters_out) iters_out[s] = stat[s].m;
    if (eps_out) eps_out[s] = stat[s].eps;
  }
  return lanczos_status_code(ctx, stat, nsys);
}

extern "C" int lanczos_sqrt_apply_multi(rpb_ctx *ctx, const rpb_params *p, int64_t n,
                                        const double *pos, int32_t nvec, const double *w,
                                        double tol, int max_iter, double *out, int *iters_out,
                                        double *eps_out, rpb_stream_t stream_) {
  RPB_TRY(check_params(ctx, p));
  if (n < 0) return fail(ctx, RPB_EINVAL, "n must be >= 0");
  if (nvec < 0 || nvec > kMaxBatchSystems)
    return fail(ctx, RPB_EINVAL, "nvec must be in [0, %d]", kMaxBatchSystems);
  if (p->lx > 0.0)
    return fail(ctx, RPB_EINVAL, "pseudo-periodic boundaries are not supported for "
                                 "multi-vector products");
  if (!(tol > 0.0)) return fail(ctx, RPB_EINVAL, "tol must be > 0");
  if (max_iter < 1 || max_iter > kMaxKrylov)
    return fail(ctx, RPB_EINVAL, "max_iter must be in [1, %d]", kMaxKrylov);
  for (int s = 0; s < nvec; ++s) {
    if (iters_out) iters_out[s] = 0;
    if (eps_out) eps_out[s] = 0.0;
  }
  if (n == 0 || nvec == 0) return RPB_OK;
  if (!pos || !w || !out) return fail(ctx, RPB_EINVAL, "pos, w and out must not be NULL");
  const size_t pb = size_t(n) * 3 * sizeof(double), vb = pb * size_t(nvec);
  if (overlaps(out, vb, pos, pb) || overlaps(out, vb, w, vb))
    return fail(ctx, RPB_EINVAL, "out overlaps an input");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  RPB_HIP(ctx, hipSetDevice(ctx->device));
  RPB_TRY(check_finite(ctx, pos, n, stream));
  // vector v is segment v of a batch of nvec segments of n spheres each
  std::vector<int64_t> offs(size_t(nvec) + 1);
  for (int s = 0; s <= nvec; ++s) offs[size_t(s)] = int64_t(s) * n;
  Batch b;
  RPB_TRY(prepare_batch(ctx, nvec, offs.data(), p->precision, &b, stream, false));
  Packed g;
  RPB_TRY(pack_geometry(ctx, p, n, pos, WS_GEOM, &g, stream));
  // Up to a few thousand spheres a product takes less than the host needs to read the flags and
  // launch the next one, so the host reads them one iteration late; a vector that has just
  // stopped then rides along in one more product (17 us of pair kernel for four vectors at 1,100
  // spheres, against ~70 us of idle device), whose launches return at once when all have.
  const int lag = n <= 4096 ? 1 : 0;
  auto product = [&](SegProduct &job, double *u) {
    return matvec_multi(ctx, p, g, nvec, job.done_host, job.vk, u, stream, &job.dot,
                        job.done_dev + nvec);
  };
  LzStatus *stat = static_cast<LzStatus *>(host_scratch(ctx));
  RPB_TRY(lanczos_segments(ctx, b, nullptr, nullptr, w, tol, max_iter, product, nullptr, nullptr,
                           p->precision == RPB_FP64, nullptr, out, true, lag, stat, stream));
  for (int s = 0; s < nvec; ++s) {
    if (iters_out) iters_out[s] = stat[s].m;
    if (eps_out) eps_out[s] = stat[s].eps;
  }
  return lanczos_status_code(ctx, stat, nvec);
}

extern "C" int lanczos_tridiag_sqrt(rpb_ctx *ctx, int32_t m, const double *alpha,
                                    const double *beta, double wnorm, double *y_out,
                                    rpb_stream_t stream_) {
  if (!ctx) return RPB_EINVAL;
  if (m < 1 || m > kMaxKrylov) return fail(ctx, RPB_EINVAL, "m must be in [1, %d]", kMaxKrylov);
  if (!alpha || (m > 1 && !beta) || !y_out)
    return fail(ctx, RPB_EINVAL, "alpha, beta and y_out must not be NULL");
  if (!std::isfinite(wnorm) || wnorm < 0.0)
    return fail(ctx, RPB_EINVAL, "wnorm must be finite and >= 0");
  LzState h{};
  for (int i = 0; i < m; ++i) {
    if (!std::isfinite(alpha[i]) || (i < m - 1 && !std::isfinite(beta[i])))
      return fail(ctx, RPB_EINVAL, "alpha and beta must be finite");
    h.alpha[i] = alpha[i];
    if (i < m - 1) h.beta[i] = beta[i];
  }
  h.wnorm = wnorm;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  RPB_HIP(ctx, hipSetDevice(ctx->device));
  int st;
  LzState *ls = static_cast<LzState *>(workspace(ctx, WS_SMALL, kSmallBytes, &st));
  if (!ls) return st;
  LzEig *eig = static_cast<LzEig *>(workspace(ctx, WS_LZEIG, sizeof(LzEig), &st));
  if (!eig) return st;
  const size_t ybytes = size_t(m) * size_t(m) * sizeof(double);
  char *buf = static_cast<char *>(workspace(ctx, WS_VEC_A, ybytes + sizeof(int), &st));
  if (!buf) return st;
  int *flag = reinterpret_cast<int *>(buf + ybytes);
  RPB_HIP(ctx, hipMemcpyAsync(ls, &h, sizeof(LzState), hipMemcpyHostToDevice, stream));
  tridiag_sequence<<<1, kThreads, 0, stream>>>(m, ls, eig, reinterpret_cast<double *>(buf), flag);
  RPB_LAUNCHED(ctx);
  int failed = 0;
  RPB_HIP(ctx, hipMemcpyAsync(y_out, buf, ybytes, hipMemcpyDeviceToHost, stream));
  RPB_HIP(ctx, hipMemcpyAsync(&failed, flag, sizeof(int), hipMemcpyDeviceToHost, stream));
  RPB_HIP(ctx, hipStreamSynchronize(stream));
  if (failed) return fail(ctx, RPB_EDEVICE, "tridiagonal eigensolve did not converge");
  return RPB_OK;
}
