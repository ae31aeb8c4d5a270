// Whole spectrum of the dense definite pencil (M, W) on many workgroups: the correlation energy of
// arXiv 2512.12515 (section "Total Energy", Eq. correlation_energy) at orders above the
// one-workgroup solver's.
//
// With 2 mu inside the gap, K = M - 2 mu W is positive definite. K z = (Omega - 2 mu) W z, so the
// eigenvalues lambda = Omega - 2 mu are those of W K = W L L^T (K = L L^T, Cholesky), which is
// similar to the symmetric S = L^T W L; lambda > 0 exactly for the pp roots (z^T K z > 0 and
// lambda z^T W z = z^T K z). The steps:
//   1. K = M - 2 mu W;
//   2. K = L L^T by the blocked right-looking Cholesky: a one-workgroup factorisation of each
//      32 x 32 diagonal block, the panel below it by forward substitution (a row per thread),
//      the trailing lower triangle updated in 32 x 32 tiles;
//   3. S = L^T W L in 32 x 32 tiles (both triangles written);
//   4. Householder reduction of S to tridiagonal form, one reflection per column: the reflection
//      vector (one workgroup), p = beta S2 v (a wave per row), then S2 -= v w^T + w v^T with
//      w = p - (beta p^T v / 2) v (every workgroup forms the dot product itself, in the same fixed
//      order);
//   5. every eigenvalue of the tridiagonal form by Sturm-count bisection (a thread per
//      eigenvalue), and the sums of the sum rule in a fixed order.
// The direct solve for the wanted roots (Eq. eigen_equation with the normalisation of Eq.
// xy_norm) runs steps 1-4 keeping the reflection vectors, then
//   5'. the wanted eigenvalues only: the Sturm count at 0 gives the number of hh roots, and
//      multisection (a workgroup per root, 256 Sturm counts per round) the j-th eigenvalue above
//      (pp) or below (hh) 0;
//   6. their eigenvectors u of the tridiagonal form by inverse iteration (a thread per root),
//      orthonormalised among nearly equal eigenvalues;
//   7. per root (a workgroup each, the vector in LDS): the reflections applied to u, then
//      L^T z = u by blocked back substitution and z scaled by sqrt|lambda|, so that
//      z^T W z = |lambda| u^T S^-1 u = sign(lambda) (S^-1 = L^-1 W L^-T).
// Every reduction runs in a fixed order: the result is bitwise repeatable.
#include <algorithm>

#include "internal.h"
#include "wave.h"

namespace pprpa {
namespace {

constexpr int CB = 32;  // Cholesky block and tile edge

// sum over the workgroup (every thread gets it); red: blockDim.x / 64 doubles of LDS
__device__ __forceinline__ double wg_sum(double v, double* red) {
  v = wave_total(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r += red[w];
  __syncthreads();
  return r;
}

__device__ __forceinline__ double wg_max(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, red[w]);
  __syncthreads();
  return r;
}

__device__ __forceinline__ double wg_min(double v, double* red) {
  return -wg_max(-v, red);
}

// (row, col) of pair index x in the lower triangle of a t x t tile grid (row >= col)
__device__ __forceinline__ void tri_pair(int x, int* r, int* c) {
  int i = (int)((sqrt(8.0 * x + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= x) ++i;
  while (i * (i + 1) / 2 > x) --i;
  *r = i;
  *c = x - i * (i + 1) / 2;
}

__global__ void k_mw_init(int* flag, int* lost) {
  if (threadIdx.x == 0) flag[0] = lost[0] = 0;
}

// K = M - mu2 W, mu2 = 2 mu, W = diag(+1 for i < nvv, -1)
__global__ __launch_bounds__(256) void k_mw_shift(const double* __restrict__ M, int n, int64_t nvv,
                                                  double mu2, double* __restrict__ K) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int i = (int)(e / n), j = (int)(e % n);
  K[e] = M[e] - (i == j ? mu2 * (i < nvv ? 1.0 : -1.0) : 0.0);
}

// Cholesky of the diagonal block at (j0, j0) (b = min(CB, n - j0) rows, lower) and the panel below
// it: row i >= j0 + CB solves x L_jj^T = K[i][j0 .. j0 + CB) by forward substitution, a row per
// thread. Every workgroup factorises the block itself (wave 0, a row per lane, columns in
// registers, the pivot column broadcast by lane reads: with the panel 14 us, against 22 for the block
// in LDS with three barriers a column and 9 for the panel in a launch of its own), workgroup 0 writes it to D (CB x CB, row-major); the block in K is
// overwritten by the next kernel, since other workgroups still read it here. A non-positive pivot
// sets flag.
__global__ __launch_bounds__(256) void k_mw_chol_panel(double* __restrict__ K, int n, int j0,
                                                       double* __restrict__ D,
                                                       int* __restrict__ flag) {
  __shared__ double l[CB][CB + 2], inv[CB];  // l by columns
  const int b = min(CB, n - j0), t = threadIdx.x;
  if (t < 64) {
    double a[CB];
    const int r = min(t, b - 1);
#pragma unroll
    for (int c = 0; c < CB; ++c) a[c] = t < b && c <= r ? K[(int64_t)(j0 + r) * n + j0 + c] : 0.0;
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      if (c < b) {  // uniform
        const double piv = lane_value(a[c], c);
        if (!(piv > 0.0) && t == 0 && blockIdx.x == 0) flag[0] = 1;
        // 1 / sqrt by the hardware's estimate and two Newton steps
        double ic = __builtin_amdgcn_rsq(piv);
        ic = piv > 0.0 ? ic : 0.0;
        ic = ic * __builtin_fma(-0.5 * piv * ic, ic, 1.5);
        ic = ic * __builtin_fma(-0.5 * piv * ic, ic, 1.5);
        double dc = piv * ic;
        dc = __builtin_fma(__builtin_fma(-dc, dc, piv), 0.5 * ic, dc);
        if (!(piv > 0.0)) dc = 0.0;
        a[c] = t == c ? dc : (t > c ? a[c] * ic : 0.0);
        if (t == 0) inv[c] = ic;
#pragma unroll
        for (int k = c + 1; k < CB; ++k) {
          const double lk = lane_value(a[c], k);  // 0 for k >= b
          a[k] = __builtin_fma(-a[c], lk, a[k]);  // (above the diagonal: not used)
        }
      }
    }
    if (t < CB) {
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        l[c][t] = a[c];
        if (blockIdx.x == 0) D[t * CB + c] = a[c];
      }
      if (t >= b) inv[t] = 0.0;
    }
  }
  __syncthreads();
  const int i = j0 + CB + blockIdx.x * 256 + t;
  if (i >= n) return;
  double x[CB];
  double* row = K + (int64_t)i * n + j0;
#pragma unroll
  for (int c = 0; c < CB; ++c) x[c] = row[c];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    x[c] *= inv[c];
#pragma unroll
    for (int k = c + 1; k < CB; ++k) x[k] -= x[c] * l[c][k];
  }
#pragma unroll
  for (int c = 0; c < CB; ++c) row[c] = x[c];
}

// The factorised diagonal block into K (the last block, which has no panel below).
__global__ __launch_bounds__(256) void k_mw_chol_store(double* __restrict__ K, int n, int j0,
                                                       const double* __restrict__ D) {
  for (int e = threadIdx.x; e < CB * CB; e += 256) {
    const int r = e / CB, c = e % CB;
    if (j0 + r < n && c <= r) K[(int64_t)(j0 + r) * n + j0 + c] = D[e];
  }
}

// Trailing update of the lower triangle right of the panel: K[i][k] -= sum_t L[i][j0+t] L[k][j0+t]
// for j0 + CB <= k <= i, one 32 x 32 tile (I >= J) per workgroup, four elements per thread; the first
// workgroup also stores the factorised diagonal block D.
__global__ __launch_bounds__(256) void k_mw_chol_update(double* __restrict__ K, int n, int j0,
                                                        const double* __restrict__ D) {
  __shared__ double pi[CB][CB + 1], pk[CB][CB + 1];
  if (blockIdx.x == 0)
    for (int e = threadIdx.x; e < CB * CB; e += 256) {
      const int r = e / CB, c = e % CB;
      if (c <= r) K[(int64_t)(j0 + r) * n + j0 + c] = D[e];
    }
  int I, J;
  tri_pair(blockIdx.x, &I, &J);
  const int r0 = j0 + CB + I * CB, c0 = j0 + CB + J * CB;
  for (int e = threadIdx.x; e < CB * CB; e += 256) {
    const int r = e / CB, t = e % CB;
    pi[r][t] = r0 + r < n ? K[(int64_t)(r0 + r) * n + j0 + t] : 0.0;
    pk[r][t] = c0 + r < n ? K[(int64_t)(c0 + r) * n + j0 + t] : 0.0;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < CB * CB; e += 256) {
    const int r = e / CB, c = e % CB;
    const int i = r0 + r, k = c0 + c;
    if (i < n && k < n && k <= i) {
      double s = 0.0;
#pragma unroll
      for (int t = 0; t < CB; ++t) s += pi[r][t] * pk[c][t];
      K[(int64_t)i * n + k] -= s;
    }
  }
}

// S = L^T W L (L: the lower triangle of K; the entries above its diagonal are ignored), tiles
// (I, J) with I >= J, both triangles written: S[i][j] = sum over k >= max(i, j) of
// L[k][i] w_k L[k][j].
__global__ __launch_bounds__(256) void k_mw_sym(const double* __restrict__ K, int n, int64_t nvv,
                                                double* __restrict__ S) {
  __shared__ double a[CB][CB + 1], bb[CB][CB + 1];
  int I, J;
  tri_pair(blockIdx.x, &I, &J);
  const int i0 = I * CB, j0 = J * CB;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k0 = i0; k0 < n; k0 += CB) {
    __syncthreads();
    for (int e = threadIdx.x; e < CB * CB; e += 256) {
      const int kk = e / CB, c = e % CB;
      const int k = k0 + kk;
      const double w = k < nvv ? 1.0 : -1.0;
      const int ci = i0 + c, cj = j0 + c;
      a[kk][c] = (k < n && ci < n && k >= ci) ? K[(int64_t)k * n + ci] * w : 0.0;
      bb[kk][c] = (k < n && cj < n && k >= cj) ? K[(int64_t)k * n + cj] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = threadIdx.x + 256 * q;
      const int r = e / CB, c = e % CB;
      double s = acc[q];
#pragma unroll 8
      for (int kk = 0; kk < CB; ++kk) s += a[kk][r] * bb[kk][c];
      acc[q] = s;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = threadIdx.x + 256 * q;
    const int i = i0 + e / CB, j = j0 + e % CB;
    if (i < n && j < n) {
      S[(int64_t)i * n + j] = acc[q];
      S[(int64_t)j * n + i] = acc[q];
    }
  }
}

// Householder step k: x = S[k][k+1 ..] (column k below the diagonal, read as row k), alpha =
// -sign(x_0) |x|, v = x - alpha e_1, beta = 2 / v^T v (0 when x = 0); d[k] = S[k][k], e[k] = alpha.
// Launched for the first step; the update kernel of step k forms the vector of step k + 1.
__global__ __launch_bounds__(1024) void k_mw_hh_vec(const double* __restrict__ S, int n, int k,
                                                    double* __restrict__ v,
                                                    double* __restrict__ scal,
                                                    double* __restrict__ d,
                                                    double* __restrict__ e,
                                                    double* __restrict__ beta_keep) {
  __shared__ double red[16];
  const int m = n - k - 1;
  const double* x = S + (int64_t)k * n + k + 1;
  double s = 0.0;
  for (int i = threadIdx.x; i < m; i += 1024) s += x[i] * x[i];
  const double nrm2 = wg_sum(s, red);
  const double x0 = x[0];
  const double nrm = sqrt(nrm2);
  const double alpha = nrm > 0.0 ? (x0 > 0.0 ? -nrm : nrm) : 0.0;
  const double v0 = x0 - alpha;
  const double vtv = nrm2 - x0 * x0 + v0 * v0;
  for (int i = threadIdx.x; i < m; i += 1024) v[i] = i == 0 ? v0 : x[i];
  if (threadIdx.x == 0) {
    const double beta = vtv > 0.0 ? 2.0 / vtv : 0.0;
    scal[0] = beta;
    if (beta_keep) beta_keep[k] = beta;
    d[k] = S[(int64_t)k * n + k];
    e[k] = alpha;
  }
}

// p = beta S2 v, S2 = S[k+1 ..][k+1 ..]: a wave per row (lanes stride the row).
__global__ __launch_bounds__(256) void k_mw_hh_matvec(const double* __restrict__ S, int n, int k,
                                                      const double* __restrict__ v,
                                                      const double* __restrict__ scal,
                                                      double* __restrict__ p) {
  const int m = n - k - 1;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= m) return;
  const double* row = S + (int64_t)(k + 1 + r) * n + k + 1;
  double s = 0.0;
  for (int j = lane; j < m; j += 64) s += row[j] * v[j];
  s = wave_total(s);
  if (lane == 0) p[r] = scal[0] * s;
}

// S2 -= v w^T + w v^T, w = p - (beta p^T v / 2) v: a wave per row; every workgroup forms p^T v
// itself in the same fixed order. keep: row k right of the diagonal becomes the reflection vector
// (only its first entry differs from x; no kernel of this step reads row k). The wave of row
// k + 1, the first row of S2, then forms the reflection of step k + 1 from the row it has just
// updated (as k_mw_hh_vec does; its norm summed over the wave's lanes in a fixed order) into the
// other buffer of v and beta: v_next, beta_next[0], d[k + 1], e[k + 1] (and beta_keep[k + 1]).
__global__ __launch_bounds__(256) void k_mw_hh_update(double* __restrict__ S, int n, int k,
                                                      const double* __restrict__ v,
                                                      const double* __restrict__ bet,
                                                      const double* __restrict__ p, int keep,
                                                      double* __restrict__ v_next,
                                                      double* __restrict__ beta_next,
                                                      double* __restrict__ d,
                                                      double* __restrict__ e,
                                                      double* __restrict__ beta_keep) {
  __shared__ double red[4];
  if (keep && blockIdx.x == 0 && threadIdx.x == 0) S[(int64_t)k * n + k + 1] = v[0];
  const int m = n - k - 1;
  double s = 0.0;
  for (int i = threadIdx.x; i < m; i += 256) s += p[i] * v[i];
  const double ptv = wg_sum(s, red);
  const double kk = 0.5 * bet[0] * ptv;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= m) return;
  const double vr = v[r], wr = p[r] - kk * vr;
  double* row = S + (int64_t)(k + 1 + r) * n + k + 1;
  const bool next = r == 0 && k + 3 < n;  // uniform over the wave
  double ss = 0.0, x0 = 0.0, dg = 0.0;
  for (int j = lane; j < m; j += 64) {
    const double vj = v[j], wj = p[j] - kk * vj;
    const double nv = row[j] - (vr * wj + wr * vj);
    row[j] = nv;
    if (j == 0) dg = nv;
    if (j == 1) x0 = nv;
    if (j >= 1) ss += nv * nv;
  }
  if (!next) return;
  const double nrm2 = wave_total(ss);
  x0 = __shfl(x0, 1, 64);
  dg = __shfl(dg, 0, 64);
  const double nrm = sqrt(nrm2);
  const double alpha = nrm > 0.0 ? (x0 > 0.0 ? -nrm : nrm) : 0.0;
  const double v0 = x0 - alpha;
  const double vtv = nrm2 - x0 * x0 + v0 * v0;
  for (int j = lane + (lane == 0 ? 64 : 0); j < m; j += 64) v_next[j - 1] = j == 1 ? v0 : row[j];
  if (lane == 0) {
    const double beta = vtv > 0.0 ? 2.0 / vtv : 0.0;
    beta_next[0] = beta;
    if (beta_keep) beta_keep[k + 1] = beta;
    d[k + 1] = dg;
    e[k + 1] = alpha;
  }
}

// Eigenvalues of T below x: sign changes of the leading minors p_i = (d_i - x) p_{i-1} -
// e_{i-1}^2 p_{i-2}. t2: (d_i, e_{i-1}^2) of T scaled by a power of two to norm 1 .. 2 (x scaled
// alike), filled up with (4, 0), which change no sign, to a multiple of 8 and by 8 more (a block is
// read ahead). Each minor takes the sign of exact arithmetic on a T perturbed by roundings, as the
// ratios p_i / p_{i-1} do, but a step of the chain is one FMA and not a division. |p| grows by at
// most 2^3 and shrinks by at most 2^100 a step: rescaled every 8 steps. A minor of 0 may count with
// either sign, as the next one has the sign opposite to the one before it; only where the
// off-diagonal element after it is 0 as well, all that follow are 0: such a block is taken again with
// the 0 as just past the sign change.
__device__ __forceinline__ int mw_sturm_below(const double* __restrict__ t2, int n, double x) {
  double p0 = 0.0, p1 = 1.0;
  int cnt = 0;
  auto step = [&](double di, double e2) __attribute__((always_inline)) {
    const double p2 = __builtin_fma(di - x, p1, -(e2 * p0));
    cnt += (int)((unsigned)(__double2hiint(p2) ^ __double2hiint(p1)) >> 31);
    p0 = p1;
    p1 = p2;
  };
  double a[16], c[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) a[u] = t2[u];
  for (int i = 0; i < n; i += 8) {
    const double s0 = p0, s1 = p1;
    const int sc = cnt;
#pragma unroll
    for (int u = 0; u < 16; ++u) c[u] = a[u];
#pragma unroll
    for (int u = 0; u < 16; ++u) a[u] = t2[2 * i + 16 + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) step(c[2 * u], c[2 * u + 1]);
    if (p0 == 0.0 && p1 == 0.0) {
      p0 = s0;
      p1 = s1 == 0.0 ? copysign(0x1p-100, s1) : s1;
      cnt = sc;
      for (int u = i; u < i + 8; ++u) {
        step(t2[2 * u], t2[2 * u + 1]);
        if (p1 == 0.0) {
          cnt += (int)((unsigned)(__double2hiint(p1) ^ ~__double2hiint(p0)) >> 31);
          p1 = p0 * -0x1p-100;
        }
      }
    }
    const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
    p0 = ldexp(p0, -ex);
    p1 = ldexp(p1, -ex);
  }
  return cnt;
}

constexpr __host__ __device__ size_t sturm_elems(int n) { return 2 * ((size_t)n + 15); }

// Matrix blockIdx.x: the last two diagonal and the last off-diagonal entry (from S, if given), then the Gershgorin interval of T:
// bnd[0] = lower, bnd[1] = upper, bnd[2] = a norm of T, and t2: T
// scaled by bnd[3], a power of two, as mw_sturm_below takes it.
__global__ __launch_bounds__(1024) void k_mw_bounds(const double* __restrict__ S, int n,
                                                    double* __restrict__ d, double* __restrict__ e,
                                                    double* __restrict__ bnd,
                                                    double* __restrict__ t2) {
  __shared__ double red[16];
  d += (size_t)blockIdx.x * n;
  e += (size_t)blockIdx.x * n;
  bnd += blockIdx.x * 4;
  t2 += blockIdx.x * sturm_elems(n);
  if (S && threadIdx.x == 0) {
    if (n >= 2) {
      d[n - 2] = S[(int64_t)(n - 2) * n + n - 2];
      e[n - 2] = S[(int64_t)(n - 1) * n + n - 2];
    }
    d[n - 1] = S[(int64_t)(n - 1) * n + n - 1];
  }
  __syncthreads();
  double lo = 1e300, hi = -1e300, nr = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
    nr = fmax(nr, fabs(d[i]) + r);
  }
  const double glo = wg_min(lo, red), ghi = wg_max(hi, red), gn = wg_max(nr, red);
  if (threadIdx.x == 0) {
    bnd[0] = glo;
    bnd[1] = ghi;
    bnd[2] = fmax(gn, 1e-300);
  }
  int ex = 0;
  frexp(fmin(fmax(gn, 1e-300), 1e300), &ex);
  const double sc = ldexp(1.0, 1 - ex);
  if (threadIdx.x == 0) bnd[3] = sc;
  for (int i = threadIdx.x; i < (n + 15) / 8 * 8; i += 1024) {
    const double ei = i > 0 && i < n ? e[i - 1] * sc : 0.0;
    t2[2 * i] = i < n ? d[i] * sc : 4.0;
    t2[2 * i + 1] = ei * ei;
  }
}

// Eigenvalue idx (ascending) of T, L lanes each: per round the lanes take the Sturm count at L
// evenly spaced interior points of the bracket, which shrinks to the two neighbouring points that
// enclose the index (reduced over the lanes by shuffles), until its width is at the rounding level.
// A wave runs until its brackets are done. A whole wave an eigenvalue (9 rounds instead of 13) as
// long as their waves fit the chip together (n <= 4096). n = 1071: 0.32 ms, against 1.43 with 16
// lanes and the ratios' divisions.
// DOWN: the eigenvalues of matrix blockIdx.y, descending and clamped at zero.
template <int L, bool DOWN>
__global__ __launch_bounds__(256) void k_mw_bisect(const double* __restrict__ t2, int n,
                                                   const double* __restrict__ bnd,
                                                   double* __restrict__ lam) {
  t2 += blockIdx.y * sturm_elems(n);
  bnd += blockIdx.y * 4;
  lam += (size_t)blockIdx.y * n;
  const int gid = blockIdx.x * 256 + threadIdx.x;
  const int idx = gid / L, g = gid % L;
  const double tnorm = bnd[2], sc = bnd[3];
  const double tiny = 1e-300 + 2.2e-16 * tnorm * 1e-8;
  double lo = bnd[0] - 1e-12 * tnorm, hi = bnd[1] + 1e-12 * tnorm;
  bool done = idx >= n;
  for (int round = 0; round < 64; ++round) {
    if (!done) done = !(hi - lo > 4.4e-16 * fmax(fabs(lo), fabs(hi)) + tiny);
    if (__all(done)) break;
    const double x = lo + (hi - lo) * ((double)(g + 1) / (L + 1.0));
    double xl = -1e300, xh = 1e300;
    if (!done && x > lo && x < hi) {
      if (mw_sturm_below(t2, n, x * sc) <= idx)
        xl = x;
      else
        xh = x;
    }
    for (int off = L / 2; off > 0; off >>= 1) {
      xl = fmax(xl, __shfl_xor(xl, off, 64));
      xh = fmin(xh, __shfl_xor(xh, off, 64));
    }
    if (!done) {
      const double nlo = fmax(lo, xl), nhi = fmin(hi, xh);
      // (counts out of order lie within their rounding of the eigenvalue: it is between the two points)
      done = nlo >= nhi || (nlo == lo && nhi == hi);
      lo = fmin(nlo, nhi);
      hi = fmax(nlo, nhi);
    }
  }
  const double mid = 0.5 * (lo + hi);
  if (idx < n && g == 0) lam[DOWN ? n - 1 - idx : idx] = DOWN ? fmax(mid, 0.0) : mid;
}

// out[0] = sum over lambda > 0 of (mu2 + lambda) - Tr A, out[1] = -(sum over lambda < 0 of
// (mu2 + lambda)) - Tr C, out[2] = Tr A, out[3] = Tr C; info: [0] 0 / 1 (K not positive definite),
// [1] pp roots, [2] hh roots. Fixed-order sums (one workgroup).
__global__ __launch_bounds__(1024) void k_mw_sums(const double* __restrict__ M, int n,
                                                  int64_t nvv, double mu2,
                                                  const double* __restrict__ lam,
                                                  const int* __restrict__ flag,
                                                  double* __restrict__ out,
                                                  int* __restrict__ info) {
  __shared__ double red[16];
  double spp = 0.0, shh = 0.0, npp = 0.0, nhh = 0.0, tra = 0.0, trc = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) {
    const double l = lam[i], om = mu2 + l;
    if (l > 0.0) {
      spp += om;
      npp += 1.0;
    } else {
      shh += om;
      nhh += 1.0;
    }
    if (i < nvv)
      tra += M[(int64_t)i * n + i];
    else
      trc += M[(int64_t)i * n + i];
  }
  const double SPP = wg_sum(spp, red), SHH = wg_sum(shh, red);
  const double NPP = wg_sum(npp, red), NHH = wg_sum(nhh, red);
  const double TA = wg_sum(tra, red), TC = wg_sum(trc, red);
  if (threadIdx.x == 0) {
    out[0] = SPP - TA;
    out[1] = -SHH - TC;
    out[2] = TA;
    out[3] = TC;
    info[0] = info[1] ? 4 : (flag[0] ? 1 : 0);  // (info[1]: the reduction's lost flag, until here)
    info[1] = (int)NPP;
    info[2] = (int)NHH;
  }
}

// Ascending index of wanted root j: pp (channel 0) the j-th eigenvalue above 0, hh the j-th below
// 0; -1 when the channel has no such root.
__device__ __forceinline__ int mw_wanted(int j, int nbelow, int n, int channel) {
  const int idx = channel == 0 ? nbelow + j : nbelow - 1 - j;
  return idx >= 0 && idx < n ? idx : -1;
}

// Wanted eigenvalue j of T (a workgroup each): per round the 256 threads take the Sturm count at
// 256 evenly spaced interior points of the bracket, which shrinks to the two neighbouring points
// that enclose the root's index, until its width is at the rounding level. lam[j] = 0 for a root
// the channel does not have.
__global__ __launch_bounds__(256) void k_mw_select(const double* __restrict__ t2, int n,
                                                   const double* __restrict__ bnd,
                                                   int* __restrict__ cnt, int channel,
                                                   const int* __restrict__ flag,
                                                   double* __restrict__ lam) {
  __shared__ double red[4];
  const int j = blockIdx.x, t = threadIdx.x;
  // eigenvalues below 0 (the hh roots)
  const int nbelow = mw_sturm_below(t2, n, 0.0);
  if (j == 0 && t == 0) cnt[0] = nbelow;
  const int idx = mw_wanted(j, nbelow, n, channel);
  if (flag[0] || idx < 0) {
    if (t == 0) lam[j] = 0.0;
    return;
  }
  const double tnorm = bnd[2], sc = bnd[3];
  const double tiny = 1e-300 + 2.2e-16 * tnorm * 1e-8;
  double lo = bnd[0] - 1e-12 * tnorm, hi = bnd[1] + 1e-12 * tnorm;
  for (int round = 0; round < 64; ++round) {
    if (!(hi - lo > 4.4e-16 * fmax(fabs(lo), fabs(hi)) + tiny)) break;
    const double x = lo + (hi - lo) * ((double)(t + 1) / 257.0);
    double xl = -1e300, xh = 1e300;
    if (x > lo && x < hi) {
      if (mw_sturm_below(t2, n, x * sc) <= idx)
        xl = x;
      else
        xh = x;
    }
    const double nlo = fmax(lo, wg_max(xl, red));
    const double nhi = fmin(hi, wg_min(xh, red));
    // (counts out of order lie within their rounding of the eigenvalue: it is between the two points, and
    // the bracket before, up to 257 times as wide, is off by as much)
    const bool last = nlo >= nhi || (nlo == lo && nhi == hi);
    lo = fmin(nlo, nhi);
    hi = fmax(nlo, nhi);
    if (last) break;
  }
  if (t == 0) lam[j] = 0.5 * (lo + hi);
}

// Eigenvector of T at lam[j] by inverse iteration (lane j): three solves of (T - lam I) y = b by
// Gaussian elimination with partial pivoting (the fill-in on a second superdiagonal), y normalised
// after each; the start vector a fixed pseudo-random sequence per root. The elimination's rows and
// the vectors are kept lane-fastest (W [4][n][64]: inverse pivots, the two superdiagonals, y), so
// that each step is one line, and a step's only division is its pivot's (a row per root and a
// division in each substitution step took 391 us at n = 225). Y [nsel][n] gets the vectors (zero
// for a root the channel does not have).
__global__ __launch_bounds__(64) void k_mw_inviter(const double* __restrict__ d,
                                                   const double* __restrict__ e, int n,
                                                   const double* __restrict__ bnd,
                                                   const int* __restrict__ cnt, int channel,
                                                   const int* __restrict__ flag,
                                                   const double* __restrict__ lam, int nsel,
                                                   double* __restrict__ Y,
                                                   double* __restrict__ W) {
  const int j = threadIdx.x;
  const bool has = j < nsel && !flag[0] && mw_wanted(j, cnt[0], n, channel) >= 0;
  double* I0 = W + j;
  double* U1 = I0 + (size_t)64 * n;
  double* U2 = U1 + (size_t)64 * n;
  double* y = U2 + (size_t)64 * n;
  const double th = has ? lam[j] : 2.0 * bnd[2];
  const double pert = 2.2e-16 * bnd[2];
  unsigned long long h = 0xD1B54A32D192ED03ull * (unsigned long long)(j + 1);
  for (int i = 0; i < n; ++i) {
    h ^= h >> 31;
    h *= 0x9FB21C651E98DF25ull;
    h ^= h >> 29;
    y[64 * (size_t)i] = 0.5 + (double)(h >> 11) * (1.0 / 9007199254740992.0);
  }
  double scale = 1.0;  // of the last solve's y
  for (int pass = 0; pass < 3; ++pass) {
    // forward elimination: row i holds (a_d, a_u, a_u2 | rhs) after the pivots above it
    double a_d = d[0] - th, a_u = n > 1 ? e[0] : 0.0, a_u2 = 0.0, rhs = y[0] * scale;
    double nextb = n > 1 ? y[64] : 0.0;
#pragma unroll 4
    for (int i = 0; i + 1 < n; ++i) {
      const double b_l = e[i], b_d = d[i + 1] - th, b_u = i + 2 < n ? e[i + 1] : 0.0;
      const double rb = nextb * scale;
      nextb = i + 2 < n ? y[64 * (size_t)(i + 2)] : 0.0;
      const bool swap = fabs(a_d) < fabs(b_l);  // rows i and i + 1 exchanged
      const double pv = swap ? b_l : a_d;
      const double piv = fabs(pv) < pert ? (pv < 0.0 ? -pert : pert) : pv;
      const double ip = 1.0 / piv;
      const double l = (swap ? a_d : b_l) * ip;
      const double p1 = swap ? b_d : a_u, p2 = swap ? b_u : a_u2, pr = swap ? rb : rhs;
      const double s0 = swap ? a_u : b_d, s1 = swap ? a_u2 : b_u, sr = swap ? rhs : rb;
      I0[64 * (size_t)i] = ip;
      U1[64 * (size_t)i] = p1;
      U2[64 * (size_t)i] = p2;
      y[64 * (size_t)i] = pr;
      a_d = s0 - l * p1;
      a_u = s1 - l * p2;
      a_u2 = 0.0;
      rhs = sr - l * pr;
    }
    if (fabs(a_d) < pert) a_d = a_d < 0.0 ? -pert : pert;
    double y1 = 0.0, y2 = rhs / a_d, nrm2 = y2 * y2;  // y2: the element just found
    y[64 * (size_t)(n - 1)] = y2;
#pragma unroll 4
    for (int i = n - 2; i >= 0; --i) {
      const double v = (y[64 * (size_t)i] - U1[64 * (size_t)i] * y2 - U2[64 * (size_t)i] * y1) *
                       I0[64 * (size_t)i];
      y[64 * (size_t)i] = v;
      y1 = y2;
      y2 = v;
      nrm2 += v * v;
    }
    scale = 1.0 / sqrt(nrm2);
  }
  if (j >= nsel) return;
  for (int i = 0; i < n; ++i) Y[(size_t)j * n + i] = has ? y[64 * (size_t)i] * scale : 0.0;
}

// The same for n <= INVITER_LDS, a workgroup (one lane of it) per root with T, the elimination and
// the vector in LDS: the elimination runs once, the next two solves take its multipliers, and a
// step's chain is two FMAs: 87 us at n = 225 and 0.40 ms at n = 1071, against 391 us and 1.87 ms with
// the vectors in memory.
constexpr int INVITER_LDS = 2048;
__global__ __launch_bounds__(64) void k_mw_inviter_lds(const double* __restrict__ d,
                                                       const double* __restrict__ e, int n,
                                                       const double* __restrict__ bnd,
                                                       const int* __restrict__ cnt, int channel,
                                                       const int* __restrict__ flag,
                                                       const double* __restrict__ lam,
                                                       double* __restrict__ Y) {
  __shared__ double dS[INVITER_LDS], eS[INVITER_LDS], ip[INVITER_LDS], u1[INVITER_LDS],
      u2[INVITER_LDS], li[INVITER_LDS], y[INVITER_LDS];
  __shared__ unsigned char sw[INVITER_LDS];
  __shared__ double last;
  const int j = blockIdx.x, lane = threadIdx.x;
  if (flag[0] || mw_wanted(j, cnt[0], n, channel) < 0) {
    for (int i = lane; i < n; i += 64) Y[(size_t)j * n + i] = 0.0;
    return;
  }
  const double th = lam[j], pert = 2.2e-16 * bnd[2];
  for (int i = lane; i < n; i += 64) {
    dS[i] = d[i] - th;
    eS[i] = i + 1 < n ? e[i] : 0.0;
    // the start vector: a mix of root and row
    unsigned long long h = 0xD1B54A32D192ED03ull * ((unsigned long long)j * 8192 + i + 1);
    h ^= h >> 31;
    h *= 0x9FB21C651E98DF25ull;
    h ^= h >> 29;
    y[i] = 0.5 + (double)(h >> 11) * (1.0 / 9007199254740992.0);
  }
  __syncthreads();
  if (lane == 0) {
    double a_d = dS[0], a_u = eS[0], a_u2 = 0.0;
#pragma unroll 4
    for (int i = 0; i + 1 < n; ++i) {
      const double b_l = eS[i], b_d = dS[i + 1], b_u = eS[i + 1];
      const bool swap = fabs(a_d) < fabs(b_l);  // rows i and i + 1 exchanged
      const double pv = swap ? b_l : a_d;
      const double r = fast_rcp(fabs(pv) < pert ? (pv < 0.0 ? -pert : pert) : pv);
      const double l = (swap ? a_d : b_l) * r;
      const double p1 = swap ? b_d : a_u, p2 = swap ? b_u : a_u2;
      const double s0 = swap ? a_u : b_d, s1 = swap ? a_u2 : b_u;
      ip[i] = r;
      u1[i] = p1;
      u2[i] = p2;
      li[i] = l;
      sw[i] = swap;
      a_d = s0 - l * p1;
      a_u = s1 - l * p2;
      a_u2 = 0.0;
    }
    if (fabs(a_d) < pert) a_d = a_d < 0.0 ? -pert : pert;
    double scale = 1.0;
    for (int pass = 0; pass < 3; ++pass) {
      double rhs = y[0] * scale;
#pragma unroll 8
      for (int i = 0; i + 1 < n; ++i) {
        const double rb = y[i + 1] * scale, l = li[i];
        const bool swap = sw[i];
        const double pr = swap ? rb : rhs;
        y[i] = pr;
        rhs = (swap ? rhs : rb) - l * pr;
      }
      double y1 = 0.0, y2 = rhs / a_d, nrm2 = y2 * y2;
      y[n - 1] = y2;
#pragma unroll 8
      for (int i = n - 2; i >= 0; --i) {
        const double v = (y[i] - u2[i] * y1 - u1[i] * y2) * ip[i];
        y[i] = v;
        y1 = y2;
        y2 = v;
        nrm2 += v * v;
      }
      scale = 1.0 / sqrt(nrm2);
    }
    last = scale;
  }
  __syncthreads();
  for (int i = lane; i < n; i += 64) Y[(size_t)j * n + i] = y[i] * last;
}

// Vectors of nearly equal eigenvalues (|lam_i - lam_j| <= 1e-7 |T|) orthonormalised in order
// (modified Gram-Schmidt; one workgroup). Only roots the channel has take part.
__global__ __launch_bounds__(1024) void k_mw_orth(int n, const double* __restrict__ bnd,
                                                  const int* __restrict__ cnt, int channel,
                                                  const int* __restrict__ flag,
                                                  const double* __restrict__ lam, int nsel,
                                                  double* __restrict__ Y) {
  __shared__ double red[16];
  if (flag[0]) return;
  const double tol = 1e-7 * bnd[2];
  for (int j = 1; j < nsel; ++j) {
    if (mw_wanted(j, cnt[0], n, channel) < 0) break;
    double* yj = Y + (size_t)j * n;
    for (int i = 0; i < j; ++i) {
      if (fabs(lam[i] - lam[j]) > tol) continue;
      const double* yi = Y + (size_t)i * n;
      double s = 0.0;
      for (int r = threadIdx.x; r < n; r += 1024) s += yi[r] * yj[r];
      const double dot = wg_sum(s, red);
      double s2 = 0.0;
      for (int r = threadIdx.x; r < n; r += 1024) {
        const double v = yj[r] - dot * yi[r];
        yj[r] = v;
        s2 += v * v;
      }
      const double inv = 1.0 / sqrt(wg_sum(s2, red));
      for (int r = threadIdx.x; r < n; r += 1024) yj[r] *= inv;
      __syncthreads();
    }
  }
}

// Root j for n <= 64 Q, one wave each, the vector in its registers (element 64 q + lane in register
// q): u = H_0 H_1 ... H_{n-3} y (reflection k in row k of S right of the diagonal, beta[k]), L^T z =
// u from the last row up, and the outputs of k_mw_vectors. A reflection is a dot product by DPP moves
// and an update, a row of the substitution a lane read and an update, with no barrier, and the next
// rows are loaded ahead: 91 us at n = 225 against 674 with a workgroup a root (1.17 ms against 3.75
// at n = 1071, the rows' way from the last-level cache to one compute unit).
template <int Q>
__global__ __launch_bounds__(64) void k_mw_back(const double* __restrict__ K,
                                                const double* __restrict__ S,
                                                const double* __restrict__ beta, int n,
                                                const int* __restrict__ cnt, int channel,
                                                const int* __restrict__ flag,
                                                const int* __restrict__ lost,
                                                const double* __restrict__ lam,
                                                const double* __restrict__ Y, double mu2,
                                                double* __restrict__ omega,
                                                double* __restrict__ Cout, int ldc,
                                                int* __restrict__ info) {
  constexpr int AHEAD = Q <= 4 ? 8 : Q <= 20 ? 4 : 2;
  const int j = blockIdx.x, lane = threadIdx.x;
  const int bad = flag[0], nb = cnt[0];
  const int npos = bad ? 0 : (channel == 0 ? n - nb : nb);
  if (j == 0 && lane == 0) {
    info[0] = lost[0] ? 4 : (bad ? 1 : (npos < (int)gridDim.x ? 2 : 0));
    info[1] = npos;
    info[2] = 0;
  }
  if (bad || j >= npos) {
    if (lane == 0) omega[j] = 0.0;
    for (int r = lane; r < n; r += 64) Cout[(size_t)r * ldc + j] = 0.0;
    return;
  }
  const double lj = lam[j];
  if (lane == 0) omega[j] = mu2 + lj;
  const double* yj = Y + (size_t)j * n;
  double y[Q], v[AHEAD][Q], b[AHEAD];
#pragma unroll
  for (int q = 0; q < Q; ++q) y[q] = 64 * q + lane < n ? yj[64 * q + lane] : 0.0;
  auto refl = [&](int k, double (&vk)[Q], double& bk) __attribute__((always_inline)) {
    bk = k >= 0 ? beta[k] : 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int r = 64 * q + lane;
      vk[q] = k >= 0 && r > k && r < n ? S[(size_t)k * n + r] : 0.0;
    }
  };
#pragma unroll
  for (int a = 0; a < AHEAD; ++a) refl(n - 3 - a, v[a], b[a]);
  for (int k = n - 3; k >= 0; k -= AHEAD) {
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) {  // (past reflection 0: zero vectors)
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) s += v[a][q] * y[q];
      const double bs = b[a] * wave_total(s);
#pragma unroll
      for (int q = 0; q < Q; ++q) y[q] -= bs * v[a][q];
      refl(k - a - AHEAD, v[a], b[a]);
    }
  }
#pragma unroll
  for (int jq = Q - 1; jq >= 0; --jq) {  // rows 64 jq + 63 .. 64 jq
    if (64 * jq >= n) continue;          // uniform
    auto row = [&](int l, double (&vk)[Q]) __attribute__((always_inline)) {
      const int c = 64 * jq + l;
#pragma unroll
      for (int q = 0; q <= jq; ++q)
        vk[q] = l >= 0 && 64 * q + lane < c ? K[(size_t)c * n + 64 * q + lane] : 0.0;
    };
    const int l0 = min(63, n - 1 - 64 * jq);
    const size_t rr = 64 * jq + min(lane, l0);
    const double dinv = 1.0 / K[rr * n + rr];
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) row(l0 - a, v[a]);
    for (int l1 = l0; l1 >= 0; l1 -= AHEAD) {
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) {
        const int l = l1 - a;
        if (l >= 0) {  // uniform
          const double z = lane_value(y[jq] * dinv, l);
#pragma unroll
          for (int q = 0; q <= jq; ++q) y[q] -= v[a][q] * z;
          y[jq] = lane == l ? z : y[jq];
        }
        row(l - AHEAD, v[a]);
      }
    }
  }
  const double sc = sqrt(fabs(lj));
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (64 * q + lane < n) Cout[(size_t)(64 * q + lane) * ldc + j] = y[q] * sc;
}

// Root j (a workgroup each; the vector in LDS, element r owned by thread r mod 256): u = H_0 H_1
// ... H_{n-3} y (reflection k kept in row k of S right of the diagonal, beta[k]), then L^T z = u
// by back substitution in 32-row blocks (the block's triangle within one wave, the rows above it
// updated by all threads), z scaled by sqrt|lambda| into column j of Cout [n][ldc]. omega[j] =
// mu2 + lambda_j; a root the channel does not have gets omega 0 and a zero column. info (block 0):
// [0] 0 ok / 1 not definite / 2 fewer than nroot roots, [1] roots of the channel, [2] 0.
__global__ __launch_bounds__(256) void k_mw_vectors(const double* __restrict__ K,
                                                    const double* __restrict__ S,
                                                    const double* __restrict__ beta, int n,
                                                    const int* __restrict__ cnt, int channel,
                                                    const int* __restrict__ flag,
                                                    const int* __restrict__ lost,
                                                    const double* __restrict__ lam,
                                                    const double* __restrict__ Y, double mu2,
                                                    double* __restrict__ omega,
                                                    double* __restrict__ Cout, int ldc,
                                                    int* __restrict__ info) {
  __shared__ double y[DENSE_SOLVE_MAX];
  __shared__ double red[2][4];
  const int j = blockIdx.x, t = threadIdx.x;
  const int bad = flag[0];
  const int nb = cnt[0];
  const int npos = bad ? 0 : (channel == 0 ? n - nb : nb);
  if (j == 0 && t == 0) {
    info[0] = lost[0] ? 4 : (bad ? 1 : (npos < (int)gridDim.x ? 2 : 0));
    info[1] = npos;
    info[2] = 0;
  }
  if (bad || j >= npos) {
    if (t == 0) omega[j] = 0.0;
    for (int r = t; r < n; r += 256) Cout[(size_t)r * ldc + j] = 0.0;
    return;
  }
  const double lj = lam[j];
  if (t == 0) omega[j] = mu2 + lj;
  for (int r = t; r < n; r += 256) y[r] = Y[(size_t)j * n + r];
  // reflections, last first; each thread updates only the elements it owns (r = t + 256 q), so
  // one barrier (inside the reduction, its partials alternating between two buffers) per
  // reflection; the next reflection's entries are loaded into registers a step ahead
  constexpr int NQ = DENSE_SOLVE_MAX / 256;
  double vc[NQ], vn[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int r = t + 256 * q;
    vc[q] = n >= 3 && r > n - 3 && r < n ? S[(size_t)(n - 3) * n + r] : 0.0;
  }
  int ph = 0;
  for (int k = n - 3; k >= 0; --k) {
    const double b = beta[k];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int r = t + 256 * q;
      vn[q] = k >= 1 && r > k - 1 && r < n ? S[(size_t)(k - 1) * n + r] : 0.0;
    }
    if (b != 0.0) {  // uniform
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int r = t + 256 * q;
        if (r > k && r < n) s += vc[q] * y[r];
      }
      s = wave_total(s);
      double* rb = red[ph];
      ph ^= 1;
      if ((t & 63) == 0) rb[t >> 6] = s;
      __syncthreads();
      const double bs = b * (rb[0] + rb[1] + rb[2] + rb[3]);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int r = t + 256 * q;
        if (r > k && r < n) y[r] -= bs * vc[q];
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) vc[q] = vn[q];
  }
  __syncthreads();
  // L^T z = u, blocks of 32 rows from the last; lane l of wave 0 holds column l of the block's
  // triangle in registers before the block's chain of shuffles
  for (int j0 = ((n - 1) / CB) * CB; j0 >= 0; j0 -= CB) {
    const int jb = min(CB, n - j0);
    if (t < 64) {
      const int l = t;
      double lc[CB];
#pragma unroll
      for (int jj = 0; jj < CB; ++jj)
        lc[jj] = jj < jb && l <= jj ? K[(size_t)(j0 + jj) * n + j0 + l] : 0.0;
      double r = l < jb ? y[j0 + l] : 0.0;
#pragma unroll
      for (int jj = CB - 1; jj >= 0; --jj) {
        if (jj < jb) {  // uniform
          const double z = l == jj ? r / lc[jj] : 0.0;
          const double zj = __shfl(z, jj, 64);
          if (l == jj) r = zj;
          if (l < jj) r -= lc[jj] * zj;
        }
      }
      if (l < jb) y[j0 + l] = r;
    }
    __syncthreads();
    for (int r = t; r < j0; r += 256) {
      double acc = 0.0;
      for (int jj = 0; jj < jb; ++jj) acc += K[(size_t)(j0 + jj) * n + r] * y[j0 + jj];
      y[r] -= acc;
    }
    __syncthreads();
  }
  const double sc = sqrt(fabs(lj));
  for (int r = t; r < n; r += 256) Cout[(size_t)r * ldc + j] = y[r] * sc;
}

}  // namespace

// Steps 1-4 (K, its Cholesky factor, S = L^T W L, the tridiagonal form (d, e) with the bounds
// of its spectrum) on stream s. v2: 2 n (the reflection vectors of two steps), bsc: 5 doubles
// ([0], [1] beta of even and odd steps, [2 .. 4] the bounds); beta_keep: n doubles or null (keep
// the reflections in the rows of S); X: tridiag_exchange(n) doubles (the tridiagonal form in one
// launch up to TRIDIAG_MAX; may overlap K where it is not needed after S), or null; flag, lost: zeroed, then set
// when K is not positive definite, or the reduction's workgroups lost one another.
static hipError_t mw_reduce(const double* M, int n, int64_t nvv, double mu2, double* K, double* S,
                            double* X, double* v2, double* p, double* d, double* e, double* bsc,
                            double* beta_keep, int* flag, int* lost, int polls, hipStream_t s) {
  const size_t nn = (size_t)n * n;
  hipLaunchKernelGGL(k_mw_init, dim3(1), dim3(64), 0, s, flag, lost);
  hipLaunchKernelGGL(k_mw_shift, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, M, n, nvv,
                     mu2, K);
  for (int j0 = 0; j0 < n; j0 += CB) {  // S, not formed yet, holds the diagonal block
    const int rest = std::max(0, n - j0 - CB);
    hipLaunchKernelGGL(k_mw_chol_panel, dim3(std::max(1, (rest + 255) / 256)), dim3(256), 0, s, K, n,
                       j0, S, flag);
    const int nt = (rest + CB - 1) / CB;
    if (rest > 0)
      hipLaunchKernelGGL(k_mw_chol_update, dim3(nt * (nt + 1) / 2), dim3(256), 0, s, K, n, j0, S);
    else
      hipLaunchKernelGGL(k_mw_chol_store, dim3(1), dim3(256), 0, s, K, n, j0, S);
  }
  const int ntile = (n + CB - 1) / CB;
  hipLaunchKernelGGL(k_mw_sym, dim3(ntile * (ntile + 1) / 2), dim3(256), 0, s, K, n, nvv, S);
  if (X && tridiag_fits(n)) {
    const hipError_t rc = launch_tridiag(S, n, 1, X, d, e, beta_keep, lost, polls, s);
    if (rc != hipSuccess) return rc;
    hipLaunchKernelGGL(k_mw_bounds, dim3(1), dim3(1024), 0, s, (const double*)nullptr, n, d, e, bsc + 2,
                       v2);
    return hipGetLastError();
  }
  if (n > 2)
    hipLaunchKernelGGL(k_mw_hh_vec, dim3(1), dim3(1024), 0, s, S, n, 0, v2, bsc, d, e, beta_keep);
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1, c = k & 1;
    double* vk = v2 + (size_t)c * n;
    double* vn = v2 + (size_t)(1 - c) * n;
    hipLaunchKernelGGL(k_mw_hh_matvec, dim3((m + 3) / 4), dim3(256), 0, s, S, n, k, vk, bsc + c, p);
    hipLaunchKernelGGL(k_mw_hh_update, dim3((m + 3) / 4), dim3(256), 0, s, S, n, k, vk, bsc + c, p,
                       beta_keep ? 1 : 0, vn, bsc + (1 - c), d, e, beta_keep);
  }
  hipLaunchKernelGGL(k_mw_bounds, dim3(1), dim3(1024), 0, s, S, n, d, e, bsc + 2, v2);
  return hipGetLastError();
}


size_t spectra_work(int n, int nmat) {
  return nmat * (tridiag_exchange(n) + 2 * (size_t)n + sturm_elems(n) + 4);
}

hipError_t launch_spectra(double* S, int n, int nmat, double* lam, double* work, int* lost,
                          int polls, hipStream_t s) {
  double* X = work;
  double* d = X + nmat * tridiag_exchange(n);
  double* e = d + (size_t)nmat * n;
  double* t2 = e + (size_t)nmat * n;
  double* bnd = t2 + nmat * sturm_elems(n);
  const hipError_t rc = launch_tridiag(S, n, nmat, X, d, e, nullptr, lost, polls, s);
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(k_mw_bounds, dim3(nmat), dim3(1024), 0, s, (const double*)nullptr, n, d, e, bnd, t2);
  hipLaunchKernelGGL((k_mw_bisect<64, true>), dim3((unsigned)((n + 3) / 4), nmat), dim3(256), 0, s, t2,
                     n, bnd, lam);
  return hipGetLastError();
}

hipError_t launch_pencil_energy_mw(const double* M, int n, int64_t nvv, double mu2, double* out,
                                   double* work, int* info, int polls, hipStream_t s) {
  if (n < 32 || n > DENSE_ENERGY_MAX) return hipErrorInvalidValue;
  const size_t nn = (size_t)n * n;
  double* S = work;
  double* v2 = S + nn;  // with p, from k_mw_bounds on: 2 (n + 15) elements
  double* p = v2 + 2 * (size_t)n;
  double* d = p + n;
  double* e = d + n;
  double* lam = e + n;
  double* bsc = lam + n;  // [0], [1] beta, [2 .. 4] Gershgorin bounds and norm
  double* K = bsc + 8;    // and, once S is formed, with the rest of work the exchange buffer
  double* X = polls >= 0 && K + tridiag_exchange(n) <= work + 3 * nn ? K : nullptr;
  int* flag = info;  // info[0], info[1] double as the flags until the last kernel
  const hipError_t rc = mw_reduce(M, n, nvv, mu2, K, S, X, v2, p, d, e, bsc, nullptr, flag, info + 1,
                                  polls, s);
  if (rc != hipSuccess) return rc;
  if (n <= 4096)
    hipLaunchKernelGGL((k_mw_bisect<64, false>), dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, v2, n,
                       bsc + 2, lam);
  else
    hipLaunchKernelGGL((k_mw_bisect<16, false>), dim3((unsigned)((n + 15) / 16)), dim3(256), 0, s, v2, n,
                       bsc + 2, lam);
  hipLaunchKernelGGL(k_mw_sums, dim3(1), dim3(1024), 0, s, M, n, nvv, mu2, lam, flag, out, info);
  return hipGetLastError();
}

size_t direct_pencil_mw_work(int n, int nroot) {
  return (n <= TRIDIAG_MAX ? tridiag_exchange(n) : 0) + 2 * (size_t)n * n + 6 * (size_t)n + (size_t)nroot * n +
         256 * (size_t)n + 64 + 8 + 8;
}

hipError_t launch_direct_pencil_mw(const double* M, int n, int64_t nvv, double mu2, int nroot,
                                   int channel, double* omega, double* Cout, int ldc,
                                   double* work, int* info, int polls, hipStream_t s) {
  if (n < 32 || n > DENSE_SOLVE_MAX || nroot < 1 || nroot > 64 || nroot > n || ldc < nroot ||
      (channel != 0 && channel != 1))
    return hipErrorInvalidValue;
  const size_t nn = (size_t)n * n;
  double* K = work;
  double* S = K + nn;
  double* X = n <= TRIDIAG_MAX ? S + nn : nullptr;
  double* v2 = S + nn + (X ? tridiag_exchange(n) : 0);
  double* p = v2 + 2 * (size_t)n;
  double* d = p + n;
  double* e = d + n;
  double* beta = e + n;
  double* Y = beta + n;
  double* W = Y + (size_t)nroot * n;
  double* lam = W + 256 * (size_t)n;  // 64
  double* bsc = lam + 64;             // [0], [1] beta, [2 .. 4] bounds
  int* cnt = (int*)(bsc + 8);         // [0] eigenvalues below 0
  int* flag = cnt + 1;                // K not positive definite
  int* lost = cnt + 2;                // the reduction's workgroups lost one another
  const hipError_t rc = mw_reduce(M, n, nvv, mu2, K, S, polls >= 0 ? X : nullptr, v2, p, d, e, bsc,
                                  beta, flag, lost, polls, s);
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(k_mw_select, dim3(nroot), dim3(256), 0, s, v2, n, bsc + 2, cnt, channel, flag,
                     lam);
  if (n <= INVITER_LDS)
    hipLaunchKernelGGL(k_mw_inviter_lds, dim3(nroot), dim3(64), 0, s, d, e, n, bsc + 2, cnt, channel,
                       flag, lam, Y);
  else
    hipLaunchKernelGGL(k_mw_inviter, dim3(1), dim3(64), 0, s, d, e, n, bsc + 2, cnt, channel, flag,
                       lam, nroot, Y, W);
  hipLaunchKernelGGL(k_mw_orth, dim3(1), dim3(1024), 0, s, n, bsc + 2, cnt, channel, flag, lam,
                     nroot, Y);
  // one wave a root as long as its vector and the rows ahead fit the registers
  if (n <= 64 * 4)
    hipLaunchKernelGGL(k_mw_back<4>, dim3(nroot), dim3(64), 0, s, K, S, beta, n, cnt, channel, flag,
                       lost, lam, Y, mu2, omega, Cout, ldc, info);
  else if (n <= 64 * 17)
    hipLaunchKernelGGL(k_mw_back<17>, dim3(nroot), dim3(64), 0, s, K, S, beta, n, cnt, channel, flag,
                       lost, lam, Y, mu2, omega, Cout, ldc, info);
  else if (n <= 64 * 32)
    hipLaunchKernelGGL(k_mw_back<32>, dim3(nroot), dim3(64), 0, s, K, S, beta, n, cnt, channel, flag,
                       lost, lam, Y, mu2, omega, Cout, ldc, info);
  else
    hipLaunchKernelGGL(k_mw_vectors, dim3(nroot), dim3(256), 0, s, K, S, beta, n, cnt, channel, flag,
                       lost, lam, Y, mu2, omega, Cout, ldc, info);
  return hipGetLastError();
}

}  // namespace pprpa
