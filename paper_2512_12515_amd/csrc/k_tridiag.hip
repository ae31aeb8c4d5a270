// Householder reduction of symmetric matrices to tridiagonal form with the matrix kept in the
// register files of a group of workgroups (gfx950): the dense pencil's direct solve and
// correlation energy (k_dense_mw.hip) and the NTO weights (k_linalg.hip).
//
// A reduction is a chain of n - 2 steps, each a matrix-vector product and a rank-2 update of what
// is left of the matrix. As two launches a step (the form used above TRIDIAG_MAX) a step takes two
// launch latencies and reads the matrix twice from the last-level cache, 11.2 us at n = 1071. Here
// one launch holds the matrix: G workgroups of 8 waves own the rows cyclically (row r: workgroup
// r mod G, then wave and register slot), a lane holds CPL columns (c = 64 j + lane) of its wave's
// RPW rows. A step is
//   1. each wave: (S v)_r of its rows; the workgroup's p = beta S v and row k + 1 are published;
//   2. every workgroup collects all of p and that row, a thread the columns t, t + 512, ..;
//   3. w = p - (beta p^T v / 2) v, the updated row k + 1 and its norm, from which the next
//      reflection: two sums over the workgroup, the same in every workgroup;
//   4. each wave updates its rows.
// A kept reflection goes back into its row of S, which every workgroup has read by then: its rows and
// row 0 are read ahead of its piece of step 0, and the rows are stored after a step's pieces of all
// workgroups (each has a row right of row 0: there are no more workgroups than rows) have arrived.
// One exchange between the workgroups and three barriers a step. (With step 3 done whole by each
// wave, one barrier, a step was 2.5 times as long: 17 columns a lane of the same work in 8 waves.)
// The exchanged words are their own flags: the exchange buffer is filled with a bit pattern that no
// result has (a NaN of one particular payload; a result with it is stored as another NaN), a slot
// is written once per launch, by device-scope atomic stores of 8 bytes, a workgroup's p as one
// piece (1.3 us from store to all workgroups having read, 2 with p in row order), and a reader
// polls until it differs.
//
// What bounds it: latency, 2.4 us a step at n = 225 and 3.8 at n = 1071 (the exchange 1.3 and 1.9,
// the rest three sums over a wave, three barriers, a square root and a reciprocal, one after the
// other); as two launches a step 6.4 and 11.2. In all 0.54 ms and 4.07 ms, before 1.44 and 11.96;
// 6.2 us a step at n = 1989, the widest rows, before 16.8.
//
// Every wait ends: a workgroup's stores of step k depend on its own earlier steps and on the other
// workgroups' stores of steps before k only, the workgroups of a launch fit the chip at once (at
// most one per compute unit), and launches of different streams are ordered one after the other
// (launch_tridiag). A context whose stream may use only a part of the compute units does without this
// form. Several processes on one device can still each hold a part of it and wait for
// the rest: a poll that does not end within TRIDIAG_POLLS tries (some seconds) gives up, it raises the
// abort flag, which every poll reads, and the host solves again by launches a step. (With no tries at
// all every workgroup gives up at its first poll: how the tests reach that.)
#include <algorithm>
#include <mutex>

#include "internal.h"
#include "wave.h"

namespace pprpa {
namespace {

typedef unsigned long long u64;
constexpr u64 EMPTY = 0x7FF4B1DFACE50DADull;  // a NaN; no operation produces this payload
constexpr u64 OTHER_NAN = 0x7FF8000000000000ull;
constexpr double NORM2_MIN = 0x1p-960;  // squared norm below which a row counts as 0
constexpr int TW = 8;                 // waves per workgroup

__device__ __forceinline__ void publish(double* p, double v) {
  u64 b = (u64)__double_as_longlong(v);
  if (b == EMPTY) b = OTHER_NAN;
  __hip_atomic_store((u64*)p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 peek(const double* p) {
  return __hip_atomic_load((const u64*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void k_tridiag_clear(double* __restrict__ X, size_t n,
                                                       int* __restrict__ abort_flag) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    ((u64*)X)[i] = EMPTY;
  if (blockIdx.x == 0 && threadIdx.x == 0) *abort_flag = 0;
}

// Matrix blockIdx.x / G of S [..][n][n] (both triangles), exchange buffer X [..][ldx];
// d, e [..][n]; keep (one matrix): reflection k's vector is left in row k of S right of the
// diagonal, its beta in beta_keep[k].
template <int CPL, int RPW>
__global__ __launch_bounds__(64 * TW, 2) void k_tridiag(double* __restrict__ Sall, int n, int G,
                                                        double* __restrict__ Xall, size_t ldx,
                                                        double* __restrict__ dall,
                                                        double* __restrict__ eall,
                                                        double* __restrict__ beta_keep,
                                                        int* __restrict__ abort_flag, int polls) {
  constexpr int N = 64 * CPL, NT = 64 * TW, E = (N + NT - 1) / NT, RPG = TW * RPW;
  // x: the next reflection's vector but for its first element (by parity of the step); bc: p and v
  // at k + 1, x at k + 2
  __shared__ double xS[2][N], wS[N], sumS[RPG], part[2][TW], bc[3];
  __shared__ int dead;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int mat = blockIdx.x / G, g = blockIdx.x - mat * G;
  double* __restrict__ S = Sall + (size_t)mat * n * n;
  double* X = Xall + mat * ldx;
  double* __restrict__ d = dall + (size_t)mat * n;
  double* __restrict__ e = eall + (size_t)mat * n;
  const bool lead = g == 0 && t == 0;
  if (t == 0) dead = 0;

  // row of slot i of this wave: (i TW + w) G + g
  double A[RPW][CPL], v[CPL];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int r = (i * TW + w) * G + g;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int c = 64 * j + lane;
      A[i][j] = r < n && c < n ? S[(size_t)r * n + c] : 0.0;
    }
  }
  // this thread's columns c = t + NT q: v there, and the place of p in a step's pieces
  double vo[E];
  int at[E];
  double s2 = 0.0;
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int c = t + NT * q;
    const double x = c >= 1 && c < n ? S[c] : 0.0;
    at[q] = min(c, n - 1) % G * RPG + min(c, n - 1) / G;
    vo[q] = x;
    if (c < N) xS[1][c] = x;
    s2 += x * x;
    if (c == 1) bc[2] = x;
  }
  s2 = wave_total(s2);
  if (lane == 0) part[1][w] = s2;
  if (lead) d[0] = S[0];
  __syncthreads();

  // owners (workgroup, wave, slot) of rows k and k + 1, stepped along with k; k = -1: the first
  // reflection
  int g0 = 0, q0 = 0, g1 = 1 % G, q1 = 1 / G;
  double vfirst = 0.0, beta = 0.0;  // of the current reflection
  for (int k = 0; k + 2 < n; ++k) {
    const int par = k & 1, m = n - 1 - k, j0 = (k + 1) >> 6;
    // the reflection of row k: x in xS[par ^ 1] (columns k + 1 ..), its norm's parts, x at k + 1
    double nrm2 = 0.0;
#pragma unroll
    for (int i = 0; i < TW; ++i) nrm2 += part[1][i];
    // |x| (square root by the hardware's estimate of 1 / sqrt and Newton steps), beta = 2 / v^T v =
    // 1 / (|x|^2 + |x_0| |x|)
    const double x0 = bc[2];
    double rs = __builtin_amdgcn_rsq(nrm2);
    rs = rs * __builtin_fma(-0.5 * nrm2 * rs, rs, 1.5);
    rs = rs * __builtin_fma(-0.5 * nrm2 * rs, rs, 1.5);
    double nrm = nrm2 * rs;
    nrm = __builtin_fma(__builtin_fma(-nrm, nrm, nrm2), 0.5 * rs, nrm);
    const bool some = nrm2 > NORM2_MIN;
    const double alpha = some ? (x0 > 0.0 ? -nrm : nrm) : 0.0;
    vfirst = some ? x0 - alpha : 0.0;
    beta = some ? fast_rcp(__builtin_fma(fabs(x0), nrm, nrm2)) : 0.0;
#pragma unroll
    for (int q = 0; q < E; ++q)
      if (t + NT * q == k + 1) vo[q] = vfirst;
#pragma unroll
    for (int j = 0; j < CPL; ++j) v[j] = xS[par ^ 1][64 * j + lane];
#pragma unroll
    for (int j = 0; j < CPL; ++j)
      if (j == j0) v[j] = lane == ((k + 1) & 63) ? vfirst : v[j];
    if (lead) e[k] = alpha;
    // 1. products of this wave's rows, published with row k + 1
    double* const P = X;  // a piece of RPG per workgroup, then R[c - k - 1]
    double* const R = X + G * RPG;
    X += G * RPG + m;
    if (g == g1 && w == q1 % TW) {
      const int i1 = q1 / TW;
#pragma unroll
      for (int i = 0; i < RPW; ++i)
        if (i == i1) {
#pragma unroll
          for (int j = 0; j < CPL; ++j) {
            const int c = 64 * j + lane;
            if (c > k && c < n) publish(R + (c - k - 1), A[i][j]);
          }
        }
    }
    double s[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) s[i] = 0.0;
#pragma unroll
    for (int j = 0; j < CPL; ++j)
      if (j >= j0) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) s[i] += A[i][j] * v[j];
      }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const double sum = wave_total(s[i]);
      if (lane == 0) sumS[i * TW + w] = beta * sum;
    }
    __syncthreads();
    if (t < RPG) {
      const int r = t * G + g;
      if (r > k && r < n) publish(P + g * RPG + t, sumS[t]);
    }
    // 2. p and row k + 1 at this thread's columns
    u64 pb[E], rb[E];
    for (int tries = 1;; ++tries) {
      bool miss = polls == 0;
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const int c = t + NT * q;
        const bool in = c > k && c < n;
        pb[q] = in ? peek(P + at[q]) : 0;
        rb[q] = in ? peek(R + (c - k - 1)) : 0;
      }
#pragma unroll
      for (int q = 0; q < E; ++q) miss |= pb[q] == EMPTY || rb[q] == EMPTY;
      if (!miss) break;
      if ((tries & 1023) == 0 || polls == 0) {
        if (tries >= polls) __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          dead = 1;
          break;
        }
      }
    }
    // 3. w and the updated row k + 1 (x), its norm from column k + 2 on
    double pv = 0.0;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const double p = __longlong_as_double((long long)pb[q]);
      pv += p * vo[q];
      if (t + NT * q == k + 1) {
        bc[0] = p;
        bc[1] = vo[q];
      }
    }
    pv = wave_total(pv);
    if (lane == 0) part[0][w] = pv;
    __syncthreads();
    if (dead) return;
    pv = 0.0;
#pragma unroll
    for (int i = 0; i < TW; ++i) pv += part[0][i];
    const double kap = 0.5 * beta * pv, v1 = bc[1], w1 = bc[0] - kap * v1;
    s2 = 0.0;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int c = t + NT * q;
      const double wc = __longlong_as_double((long long)pb[q]) - kap * vo[q];
      double x = __longlong_as_double((long long)rb[q]) - (v1 * wc + w1 * vo[q]);
      if (c == k + 1 && g == 0) d[k + 1] = x;
      if (c == k + 2) bc[2] = x;
      if (c < k + 2) x = 0.0;
      s2 += x * x;
      if (c < N) {
        wS[c] = wc;
        xS[par][c] = x;
      }
      vo[q] = x;
    }
    s2 = wave_total(s2);
    if (lane == 0) part[1][w] = s2;
    __syncthreads();
    // 4. this wave's rows (wide rows: v again from LDS, its registers hold the row)
    if constexpr (CPL > 20) {
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const int r = (i * TW + w) * G + g;
        if (r > k && r < n) {
          const double vr = r == k + 1 ? vfirst : xS[par ^ 1][r], wr = wS[r];
#pragma unroll
          for (int j = 0; j < CPL; ++j)
            if (j >= j0) {
              const int c = 64 * j + lane;
              const double vc = c == k + 1 ? vfirst : xS[par ^ 1][c];
              A[i][j] -= vr * wS[c] + wr * vc;
            }
        }
      }
    } else {
      double wv[CPL];
#pragma unroll
      for (int j = 0; j < CPL; ++j) wv[j] = wS[64 * j + lane];
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const int r = (i * TW + w) * G + g;
        if (r > k && r < n) {
          const double vr = r == k + 1 ? vfirst : xS[par ^ 1][r], wr = wS[r];
#pragma unroll
          for (int j = 0; j < CPL; ++j)
            if (j >= j0) A[i][j] -= vr * wv[j] + wr * v[j];
        }
      }
    }
    // The kept reflection into row k of S. Not before the step's exchange: every workgroup takes the
    // first reflection from row 0 of S when it starts, which may be late, and has done so when its
    // piece of step 0 is there. (Rows from 1 on are read by their own workgroup only.)
    if (beta_keep && g == g0 && w == q0 % TW) {
      if (lane == 0) beta_keep[k] = beta;
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        const int c = 64 * j + lane;
        if (c > k && c < n) S[(size_t)k * n + c] = c == k + 1 ? vfirst : xS[par ^ 1][c];
      }
    }
    g0 = g1;
    q0 = q1;
    if (++g1 == G) {
      g1 = 0;
      ++q1;
    }
  }
  // what is left: e[n - 2] is the last x, row n - 1 holds only its diagonal element now
  if (lead) e[n - 2] = bc[2];
  if (g == g1 && w == q1 % TW) {
    const int i1 = q1 / TW;
#pragma unroll
    for (int i = 0; i < RPW; ++i)
      if (i == i1) {
#pragma unroll
        for (int j = 0; j < CPL; ++j)
          if (64 * j + lane == n - 1) d[n - 1] = A[i][j];
      }
  }
}

// One launch at a time on a device, across streams and contexts: each waits, on the GPU, for the
// one before (two of them could otherwise each hold part of the chip and wait for the rest).
struct Gate {
  std::mutex mu;
  hipEvent_t last = nullptr;
};
constexpr int GATES = 64;
Gate g_gate[GATES];

// Workgroups per matrix at rpw rows a wave.
int groups(int n, int rpw) { return (n + TW * rpw - 1) / (TW * rpw); }

template <int CPL, int RPW>
hipError_t run(double* S, int n, int nmat, double* X, double* d, double* e, double* beta_keep,
               int* abort_flag, int polls, int cus, hipStream_t s) {
  const int G = groups(n, RPW);
  const size_t ldx = tridiag_exchange(n);
  const int batch = cus / G;  // matrices per launch
  for (int m0 = 0; m0 < nmat; m0 += batch) {
    const int nb = nmat - m0 < batch ? nmat - m0 : batch;
    const size_t off = (size_t)m0 * n;
    hipLaunchKernelGGL((k_tridiag<CPL, RPW>), dim3(nb * G), dim3(64 * TW), 0, s, S + off * n, n, G,
                       X + m0 * ldx, ldx, d + off, e + off, beta_keep, abort_flag, polls);
  }
  return hipGetLastError();
}

// Rows a wave: as few as let every matrix have its workgroups at once (a step's products and updates
// are shorter, and more workgroups exchange as fast: 4 / 2 / 1 rows 616 / 559 / 543 us at n = 225,
// 1.57 / 1.36 / 1.29 ms at 451, 5.15 / 4.64 / 4.12 at 1071), else the most. The bits are the same: a
// row's product and the sums over columns do not depend on it.
template <int CPL, int MOST>
hipError_t run_rows(double* S, int n, int nmat, double* X, double* d, double* e, double* beta_keep,
                    int* abort_flag, int polls, int cus, hipStream_t s) {
  if ((int64_t)nmat * groups(n, 1) <= cus)
    return run<CPL, 1>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s);
  if (MOST == 2 || (int64_t)nmat * groups(n, 2) <= cus)
    return run<CPL, 2>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s);
  return run<CPL, MOST>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s);
}

}  // namespace

bool tridiag_fits(int n) {
  int dev = 0, cus = 0;
  if (n < 3 || n > TRIDIAG_MAX || hipGetDevice(&dev) != hipSuccess || dev >= GATES ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return false;
  return groups(n, n <= 512 ? 4 : n <= 1088 ? 2 : 1) <= cus;
}

// n steps' pieces of every workgroup's rows (whatever their split) and the rows.
size_t tridiag_exchange(int n) {
  return (size_t)n * (n + 4 * TW - 1) + (size_t)n * n / 2;
}

hipError_t launch_tridiag(double* S, int n, int nmat, double* X, double* d, double* e,
                          double* beta_keep, int* abort_flag, int polls, hipStream_t s) {
  int dev = 0, cus = 0;
  hipError_t rc = hipGetDevice(&dev);
  if (rc == hipSuccess) rc = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (rc != hipSuccess) return rc;
  if (!tridiag_fits(n) || nmat < 1 || polls < 0 || (beta_keep && nmat > 1)) return hipErrorInvalidValue;
  Gate& gt = g_gate[dev];
  std::lock_guard<std::mutex> lk(gt.mu);
  if (!gt.last) {
    if ((rc = hipEventCreateWithFlags(&gt.last, hipEventDisableTiming)) != hipSuccess) return rc;
  } else if ((rc = hipStreamWaitEvent(s, gt.last, 0)) != hipSuccess) {
    return rc;
  }
  const size_t total = nmat * tridiag_exchange(n), blocks = std::min<size_t>((total + 1023) / 1024, 2048);
  hipLaunchKernelGGL(k_tridiag_clear, dim3((unsigned)blocks), dim3(256), 0, s, X, total, abort_flag);
  rc = n <= 256   ? run_rows<4, 4>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s)
       : n <= 512 ? run_rows<8, 4>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s)
       : n <= 1088 ? run_rows<17, 2>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s)
                   : run<32, 1>(S, n, nmat, X, d, e, beta_keep, abort_flag, polls, cus, s);
  if (rc == hipSuccess) rc = hipEventRecord(gt.last, s);
  return rc;
}

}  // namespace pprpa
