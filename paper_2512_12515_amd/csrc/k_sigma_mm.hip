// Density-fitted sigma contraction as two matrix products (FP64 and FP32 MFMA, gfx950), for the
// restricted blocks and the alpha-beta sector:
//
//   phase 1   T[P][c][kv][col] = sum_d U_kv[c][d] Lb^P[d][col]      (every column, c's block of d)
//   phase 2   Q[kv][r][col]    = sum_{P,c} La^P[r][c] T[P][c][kv][col]   (the two diagonal blocks)
//
// (La = Lb = L and U the upper triangle of the unpacked vector, d >= c, for a restricted context;
// the method's equations and the packed layouts are those of k_sigma.hip and k_sigma_ab.hip).
// Both phases are one kind of product, C[m][n] = sum_k A[k][m] B[k][n] with A and B read as rows
// of contiguous elements (L^P is symmetric, U is stored transposed), so they share one inner loop,
// and the columns of all k vectors (phase 2) or of all P (phase 1) form one long n index: a block
// of vectors leaves no ragged column panel.
//
// Against the one-kernel forms (T in registers between the two contractions): an FP64 MFMA
// 16x16x4 takes 64 cycles, so T's way through memory (2 x 8 bytes an element, about 2 TB/s at the
// rates below, under the products) costs less than what the fused form pays for keeping T beside Q
// in registers: few row tiles a stage, a T exchange per chunk, ragged panels, 8192 and more short
// units with a partial sum each.
//   * unit: 4 waves, a panel of up to 8 row tiles by 8 column tiles (2 a wave), 16 reduction rows a
//     stage in two LDS buffers; two units a CU, whose waits the other's products cover (one
//     8-wave unit of twice the columns, or four 8-row buffers, were 5-11 % slower: more barriers);
//   * row panels are cut evenly (13 tiles: 6 + 7), each count of tiles with its own code; stages on
//     the diagonal of U skip the row tiles below it (4-6 % of phase 1 at 32 tiles, 12 % at 13);
//   * lanes read 16 bytes of LDS where they can (row tiles interleaved), a step's operands in the
//     middle of the step before; loads take a scalar base and a fixed lane offset and the LDS
//     address is scalar: 3 vector instructions a stage beside its 64 products (30 before, and each
//     costs the matrix pipe about 4 cycles: 251 -> 245 ms at 50/500/1800);
//   * phase 2 splits the aux index into slots, each with its own sums in registers over the whole
//     slot (no partial sums in between), so that the units fill whole rounds of the chip; launch c
//     runs phase 2 of part c - 1 of every slot and phase 1 of part c, whose short units fill the
//     long ones' tail. Where the workspace is small (served requests) a launch takes some slots whole
//     instead, if enough products are in it to fill the chip: the sums then stay in registers (a part of
//     one aux index reads and writes them every 9 stages at 13/117/457). FP32 sums are chains of one
//     aux index (16 times the c tiles), added up in FP64 in registers: 7.8e-8 relative error at
//     40/400/1540, against 2.3e-7 of the one-kernel form.
// What bounds it: the matrix pipe, busy 87 % of the time at 50/500/1800 (61 % before); the direct
// loads cost 6.7 %, the barriers 1.6 %, launch tails about 2 %. Times (us; 12-20 vectors):
//   FP64 50/500/1800 354518 -> 243000 (60 TFLOP/s of the 3/4 of the products the identity needs;
//   a large library product reaches 73), 20/200/700 10381 -> 7850, 13/117/457 (7 vectors) 716 -> 504;
//   FP32 40/400/1540 45015 -> 35900; alpha-beta 200/20/18 FP64 7605 -> 5870, FP32 4389 -> 3059.
//   FP64 sums are one chain a slot: the error against 64-bit references is 2.0e-15 at 50/500/1800, 9.0e-16
//   with the one-kernel form's many short sums (20/200/700 8.9e-16 and 7.3e-16).
#include "internal.h"
#include "sigma_common.h"
#include "sigma_mm.h"

namespace pprpa {
namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int MW = 4;         // waves per workgroup
constexpr int MT = MM_MT;     // row tiles per panel (accumulator rows of a wave)
constexpr int KS = TILE;      // reduction rows per stage
constexpr int NT = 2;         // column tiles per wave: one vector read of B per lane and row
constexpr int AW = MT * TILE; // row width of a staged A tile
static_assert(MW * NT == MM_BT, "column tiles of a workgroup");

template <typename T> struct Mm;
template <> struct Mm<double> {
  using Acc = d4;
};
template <> struct Mm<float> {
  using Acc = f4;
};

__device__ __forceinline__ d4 mfma_mm(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma_mm(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// A lane reads 16 contiguous bytes of a staged row where it can, so neighbouring row tiles are
// interleaved: the tiles of a panel of m form groups of 4 (FP32), 2 and 1, and element e of a
// group's vector read belongs to its tile e, i.e. tile e of a group of g tiles holds the rows
// g i + e, i = 0..15, of the group's 16 g rows.
template <typename T, int M> struct Groups {
  static constexpr int quads = sizeof(T) == 4 ? M / 4 : 0;
  static constexpr int pairs = (M - 4 * quads) / 2;
  static constexpr int ones = M & 1;
};
// Row of the panel that register j of tile m holds in lane group lk: lane_row + uniform_row (the
// MFMA's row i of register j is lk + 4 j in FP64, 4 lk + j in FP32).
template <typename T, int M> __device__ __forceinline__ int lane_row(int m, int lk) {
  using G = Groups<T, M>;
  const int i = sizeof(T) == 8 ? lk : 4 * lk;
  return m < 4 * G::quads ? 4 * i : (m < 4 * G::quads + 2 * G::pairs ? 2 * i : i);
}
template <typename T, int M> __device__ __forceinline__ int uniform_row(int m, int j) {
  using G = Groups<T, M>;
  const int i = sizeof(T) == 8 ? 4 * j : j;
  if (m < 4 * G::quads) return (m & ~3) * TILE + 4 * i + (m & 3);
  const int r = m - 4 * G::quads;
  if (r < 2 * G::pairs) return (m - (r & 1)) * TILE + 2 * i + (r & 1);
  return m * TILE + i;
}
// End of the group that starts at tile m of a panel of M.
template <typename T, int M> constexpr int group_end(int m) {
  using G = Groups<T, M>;
  return m < 4 * G::quads ? m + 4 : (m - 4 * G::quads < 2 * G::pairs ? m + 2 : m + 1);
}

template <int N> struct IntC { static constexpr int v = N; };
template <typename F> __device__ __forceinline__ void for_tiles(int m, F&& f) {
  switch (m) {
    case 1: f(IntC<1>{}); break;
    case 2: f(IntC<2>{}); break;
    case 3: f(IntC<3>{}); break;
    case 4: f(IntC<4>{}); break;
    case 5: f(IntC<5>{}); break;
    case 6: f(IntC<6>{}); break;
    case 7: f(IntC<7>{}); break;
    default: f(IntC<8>{}); break;
  }
}

template <typename T> using Lds = const __attribute__((address_space(3))) T;

template <typename T> struct Frag {
  T a[MT], b[NT];
};

// This lane's LDS byte addresses (operand reads) in the current stage buffer: the vector reads of
// 4, 2 and 1 row tiles, and the read of B.
struct LdsAt {
  Lds<char>*quad, *pair, *one, *b;
};

// One reduction step's operands (4 rows from row 4 KS of the stage) of the first G row tiles.
template <typename T, int G, int K>
__device__ __forceinline__ void read_operands(const LdsAt& at, Frag<T>& f) {
  using GG = Groups<T, G>;
  typedef T P2 __attribute__((ext_vector_type(2)));
  typedef T P4 __attribute__((ext_vector_type(4)));
  constexpr unsigned row = 4 * K * AW * sizeof(T), rowb = 4 * K * MW * NT * TILE * sizeof(T);
#pragma unroll
  for (int q = 0; q < GG::quads; ++q) {
    const P4 v = *(Lds<P4>*)(at.quad + (row + q * 4 * TILE * (unsigned)sizeof(T)));
#pragma unroll
    for (int e = 0; e < 4; ++e) f.a[4 * q + e] = v[e];
  }
#pragma unroll
  for (int p = 0; p < GG::pairs; ++p) {
    const int t = 4 * GG::quads + 2 * p;
    const P2 v = *(Lds<P2>*)(at.pair + (row + t * TILE * (unsigned)sizeof(T)));
    f.a[t] = v[0];
    f.a[t + 1] = v[1];
  }
  if (GG::ones) f.a[G - 1] = *(Lds<T>*)(at.one + (row + (G - 1) * TILE * (unsigned)sizeof(T)));
  const P2 v = *(Lds<P2>*)(at.b + rowb);
  f.b[0] = v[0];
  f.b[1] = v[1];
}

template <typename T, int M> struct Tile {
  typename Mm<T>::Acc c[M][NT];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) c[m][n] = typename Mm<T>::Acc{0, 0, 0, 0};
  }
};

// Products of row tiles [M0, M1) of one reduction step.
template <typename T, int M, int M0, int M1>
__device__ __forceinline__ void step_product(const Frag<T>& f, Tile<T, M>& acc) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int m = M0; m < M1; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc.c[m][n] = mfma_mm(f.a[m], f.b[n], acc.c[m][n]);
  __builtin_amdgcn_sched_barrier(0);
}

// One stage (KS reduction rows) of the first G row tiles of a panel of M: each step's operands are
// read from LDS in the middle of the products of the step before (the wait ahead of a step's
// products is for every outstanding LDS read, so only one step's may be in flight there).
template <typename T, int M, int G>
__device__ __forceinline__ void stage_product(const LdsAt& at, Tile<T, M>& acc) {
  static_assert(KS == 16, "four steps");
  constexpr int H = (G + 1) / 2;
  Frag<T> f[2];
  read_operands<T, G, 0>(at, f[0]);
  step_product<T, M, 0, H>(f[0], acc);
  read_operands<T, G, 1>(at, f[1]);
  step_product<T, M, H, G>(f[0], acc);
  step_product<T, M, 0, H>(f[1], acc);
  read_operands<T, G, 2>(at, f[0]);
  step_product<T, M, H, G>(f[1], acc);
  step_product<T, M, 0, H>(f[0], acc);
  read_operands<T, G, 3>(at, f[1]);
  step_product<T, M, H, G>(f[0], acc);
  step_product<T, M, 0, G>(f[1], acc);
}

// A run of stages: uniform source pointers of the next stage's first rows, stages, row tiles.
template <typename T> struct Run {
  const char* pa;
  const char* pb;
  int n, mt;
};

template <typename T> constexpr int mm_lds() {  // elements of the two stage buffers
  return 2 * KS * (AW + MW * NT * TILE);
}

// Unit idx of XCD xcd of a product's launch.
template <typename T>
__device__ __forceinline__ void mm_unit(const MmParams& p, T* buf, const int xcd, const int idx) {
  constexpr int BT = MW * NT, BW = BT * TILE, VEC = 16 / (int)sizeof(T);
  constexpr int RA = 64 * VEC / AW;         // A rows one wave load covers
  constexpr int STAGE = KS * AW + KS * BW;  // elements per stage buffer
  constexpr unsigned SB = STAGE * sizeof(T);
  constexpr int RB = 64 * VEC / BW;         // B rows one wave load covers
  static_assert(RB >= 1 && KS % (RB * MW) == 0, "whole wave loads");
  static_assert(2 * STAGE == mm_lds<T>(), "stage buffers");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  // this lane's place in an A load (row, column), in a B row and in the output columns
  const int ra = w * RA + (lane * VEC) / AW, ca = (lane * VEC) % AW;
  const int rb = w * RB + (lane * VEC) / BW;
  const int jb = (lane * VEC) % BW / TILE, cb = (lane * VEC) % TILE;
  const int js = w * NT + (NT * li) / TILE, cs = (NT * li) % TILE;

  Lds<char>* const lds0 = (Lds<char>*)(lds_ptr_t)buf;
  char __attribute__((address_space(3)))* const lds_w =
      (char __attribute__((address_space(3)))*)(lds_ptr_t)buf + w * 1024;
  unsigned cur = 0;  // byte offset of the buffer the current stage reads
  auto at = [&]() __attribute__((always_inline)) {
    Lds<char>* const row = lds0 + (cur + lk * AW * (unsigned)sizeof(T));
    constexpr unsigned b = sizeof(T);
    return LdsAt{row + 4 * li * b, row + 2 * li * b, row + li * b,
                 lds0 + (cur + (KS * AW + lk * BW + w * NT * TILE + NT * li) * b)};
  };

  unsigned va, vb;     // this lane's byte offsets from the run's pointers
  unsigned lda, ldb;   // row strides in bytes
  // direct global->LDS loads of the run's next stage into the buffer at byte offset `to`
  auto issue = [&](Run<T>& r, unsigned to) __attribute__((always_inline)) {
    char __attribute__((address_space(3)))* const b = lds_w + to;
    // (opaque 32-bit lane offsets: the loads take a scalar base and this offset, no vector
    // address arithmetic)
    asm volatile("" : "+v"(va), "+v"(vb));
    if (ca < r.mt * TILE) {
#pragma unroll
      for (int i = 0; i < KS / RA / MW; ++i)
        __builtin_amdgcn_global_load_lds((const void*)(r.pa + (size_t)(i * MW * RA) * lda + va),
                                         (lds_ptr_t)(b + i * MW * 1024), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < KS / RB / MW; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(r.pb + (size_t)(i * MW * RB) * ldb + vb),
                                       (lds_ptr_t)(b + KS * AW * sizeof(T) + i * MW * 1024), 16, 0, 0);
    r.pa += (size_t)KS * lda;
    r.pb += (size_t)KS * ldb;
  };
  // wait for the current stage's loads (this wave's, then everyone's: the barrier also means that
  // the other buffer is no longer read)
  auto arrive = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };

  if (idx < p.per2) {
    // ---- phase 2 unit: a slot (its share of the aux index), a block of columns, a row panel -----
    // (each XCD takes a contiguous run of the virtual block's units, the long ones, first; the
    // occupied block's slots are ro-ths of the virtual block's)
    const bool virt = idx < p.per2v;
    const int items = virt ? p.items2v : p.items2 - p.items2v;
    const int u = virt ? xcd * p.per2v + idx : xcd * (p.per2 - p.per2v) + idx - p.per2v;
    const int ro = virt ? 1 : p.ro;
    if (u >= items * p.slots2 * ro) return;
    const int slot = u / items, it = u - slot * items;  // of this launch
    const int sl = slot / ro, r = slot - sl * ro, s = p.slot2 + sl;
    const int lo = mm_cut(0, p.naux, p.nslot, s), hi = mm_cut(0, p.naux, p.nslot, s + 1);
    const int Plo = mm_cut(lo, hi, ro, r), Phi = mm_cut(lo, hi, ro, r + 1);
    const int Ppart = mm_cut(lo, hi, p.nparts, p.part2);
    // this launch's part of the unit's aux indices
    const int Pa = __builtin_amdgcn_readfirstlane(max(Plo, Ppart));
    const int Pb = __builtin_amdgcn_readfirstlane(min(Phi, mm_cut(lo, hi, p.nparts, p.part2 + 1)));
    if (Pa >= Pb) return;
    const int npan = virt ? p.npv : p.npo;
    const int nb = it / npan, pan = it - nb * npan;
    const int bta = virt ? p.nvta : p.ncta - p.nvta;
    const int btb = virt ? p.nvtb : p.nctb - p.nvtb;
    const int t0 = bta * pan / npan, mt = bta * (pan + 1) / npan - t0;
    const int row0 = ((virt ? 0 : p.nvta) + t0) * TILE;
    const int ctile0 = virt ? 0 : p.nvtb;
    const int ntot = p.k * btb;
    const int jl = min(nb * BT + jb, ntot - 1);
    const int jkv = jl / btb, jct = ctile0 + jl - jkv * btb;
    lda = p.nmopa * sizeof(T);
    ldb = p.k * p.nmopb * sizeof(T);
    va = ra * lda + ca * sizeof(T);
    vb = rb * ldb + (unsigned)((jkv * p.nmopb + jct * TILE + cb) * sizeof(T));
    const int jo = nb * BT + js;
    const bool store = jo < ntot;
    // this lane's part of the offsets (bytes) its results go to; the rest is uniform
    const int okv = min(jo, ntot - 1) / btb, oct = ctile0 + min(jo, ntot - 1) - okv * btb;
    const int64_t qs = virt ? p.qstride : p.qostride;
    double* const Q = virt ? p.Q : p.Qo;
    const unsigned ldq = virt ? p.nmopb : btb * TILE;
    const size_t q0 = (size_t)(p.slot2 * ro + slot) * p.k * qs + (size_t)(t0 * TILE) * ldq;
    const unsigned vq = (unsigned)(okv * qs + (oct - ctile0) * TILE + cs);
    const size_t k0 = (size_t)Pa * p.ncta * KS, kt0 = (size_t)(sl * p.mc + Pa - Ppart) * p.ncta * KS;
    Run<T> ld{(const char*)p.La + k0 * lda + row0 * sizeof(T), (const char*)p.Tin + kt0 * ldb,
              (Pb - Pa) * p.ncta, mt};
    const int n = ld.n;
    issue(ld, 0);
    for_tiles(mt, [&](auto MC) __attribute__((always_inline)) {
      constexpr int M = decltype(MC)::v;
      Tile<double, M> sum;
      sum.clear();
      // for every pair of sums of this lane: f(its place in the unit's sums, the registers, r)
      auto each = [&](auto f) __attribute__((always_inline)) {
        if (store) {
#pragma unroll
          for (int m = 0; m < M; ++m) {
            const unsigned vo = vq + lane_row<T, M>(m, lk) * ldq;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
              for (int h = 0; h < NT / 2; ++h)
                f(*(d2*)(Q + (q0 + uniform_row<T, M>(m, r) * ldq) + (vo + 2 * h)),
                  sum.c[m][2 * h], sum.c[m][2 * h + 1], r);
          }
        }
      };
      auto run_to = [&](int st, int end, auto& acc) __attribute__((always_inline)) {
        for (; st < end; ++st) {
          arrive();
          if (st + 1 < n) issue(ld, SB - cur);
          stage_product<T, M, M>(at(), acc);
          cur = SB - cur;
        }
      };
      // the sums of a unit whose aux indices come in several launches go on from one to the next
      if (Pa > Plo)
        each([&](const d2& x, d4& a, d4& b, int r) __attribute__((always_inline)) {
          a[r] = x[0];
          b[r] = x[1];
        });
      if constexpr (sizeof(T) == 8) {
        run_to(0, n, sum);
      } else {
        // FP32 chains of one aux index each (16 ncta terms), added up in FP64
        for (int st = 0; st < n; st += p.ncta) {
          Tile<T, M> acc;
          acc.clear();
          run_to(st, st + p.ncta, acc);
#pragma unroll
          for (int m = 0; m < M; ++m)
#pragma unroll
            for (int c = 0; c < NT; ++c)
#pragma unroll
              for (int r = 0; r < 4; ++r) sum.c[m][c][r] += (double)acc.c[m][c][r];
        }
      }
      each([&](d2& x, d4& a, d4& b, int r) __attribute__((always_inline)) { x = d2{a[r], b[r]}; });
    });
    return;
  }

  // ---- phase 1 unit: one vector, a block of columns of consecutive (P, column tile) -------------
  // (of one slot's aux indices in this part)
  const int u = xcd * p.per1 + idx - p.per2;
  if (u >= p.units1) return;
  const int kv = u % p.k, us = u / p.k;
  const int sl = us / p.nbs, nb = us - sl * p.nbs, s = p.slot1 + sl;
  const int lo = mm_cut(0, p.naux, p.nslot, s), hi = mm_cut(0, p.naux, p.nslot, s + 1);
  const int Ppart = mm_cut(lo, hi, p.nparts, p.part1);
  const int ntot = (mm_cut(lo, hi, p.nparts, p.part1 + 1) - Ppart) * p.nctb;
  if (nb * BT >= ntot) return;
  const int jl = min(nb * BT + jb, ntot - 1);
  const int P0 = __builtin_amdgcn_readfirstlane(nb * BT / p.nctb), jP = jl / p.nctb;
  lda = p.nmopa * sizeof(T);
  ldb = p.nmopb * sizeof(T);
  va = ra * lda + ca * sizeof(T);
  vb = rb * ldb + (unsigned)((jP - P0) * p.lbstride + (jl - jP * p.nctb) * TILE + cb) * (unsigned)sizeof(T);
  const char* const pb0 = (const char*)p.Lb + (size_t)(Ppart + P0) * p.lbstride * sizeof(T);
  const char* const pa0 = (const char*)p.UT + (size_t)kv * p.ustride * sizeof(T);
  const int jo = nb * BT + js;
  const bool store = jo < ntot;
  const int oP = min(jo, ntot - 1) / p.nctb;
  const unsigned so = p.k * p.nmopb * sizeof(T);  // row stride of T, bytes
  char* const out = (char*)p.Tout + (size_t)(sl * p.mc + P0) * p.nmopa * so + (size_t)kv * p.nmopb * sizeof(T);
  const unsigned vt = (unsigned)(oP - P0) * p.nmopa * so +
                      (unsigned)(((min(jo, ntot - 1) - oP * p.nctb) * TILE + cs) * sizeof(T));
  const int npan = p.npv + p.npo;
  // panel i: its first row tile (c), its tiles and its reduction range
  auto panel = [&](int i, int& c) __attribute__((always_inline)) {
    const bool virt = i < p.npv;
    const int np = virt ? p.npv : p.npo, j = virt ? i : i - p.npv;
    const int bt = virt ? p.nvta : p.ncta - p.nvta, base = virt ? 0 : p.nvta;
    const int t0 = __builtin_amdgcn_readfirstlane(bt * j / np);
    Run<T> r;
    c = base + t0;
    r.mt = __builtin_amdgcn_readfirstlane(bt * (j + 1) / np) - t0;
    const int dlo = p.tri ? c : (virt ? 0 : p.nvtb);
    r.n = (virt ? p.nvtb : p.nctb) - dlo;
    r.pa = pa0 + (size_t)(dlo * TILE) * lda + c * TILE * sizeof(T);
    r.pb = pb0 + (size_t)(dlo * TILE) * ldb;
    return r;
  };
  int c0;
  Run<T> ld = panel(0, c0);  // the run whose stages are being loaded, one stage ahead
  issue(ld, 0);
  for (int i = 0; i < npan; ++i) {
    const int n = ld.n, mt = ld.mt;
    int c0n = 0;
    Run<T> nx{nullptr, nullptr, 0, 0};
    if (i + 1 < npan) nx = panel(i + 1, c0n);
    for_tiles(mt, [&](auto MC) __attribute__((always_inline)) {
      constexpr int M = decltype(MC)::v;
      Tile<T, M> acc;
      acc.clear();
      int st = 0;
      auto run_to = [&](int end, auto GC) __attribute__((always_inline)) {
        for (; st < end; ++st) {
          arrive();
          if (st + 1 == n) ld = nx;  // (at the unit's end an empty run)
          if (ld.n) issue(ld, SB - cur);
          stage_product<T, M, decltype(GC)::v>(at(), acc);
          cur = SB - cur;
        }
      };
      // the stages on the diagonal of U multiply only the groups of row tiles that reach it
      // (c <= d)
      if (p.tri) {
        constexpr int e1 = group_end<T, M>(0);
        if constexpr (e1 < M) {
          run_to(min(e1, n), IntC<e1>{});
          constexpr int e2 = group_end<T, M>(e1);
          if constexpr (e2 < M) {
            run_to(min(e2, n), IntC<e2>{});
            constexpr int e3 = group_end<T, M>(e2);
            if constexpr (e3 < M) run_to(min(e3, n), IntC<e3>{});
          }
        }
      }
      run_to(n, IntC<M>{});
      if (store) {
        typedef T P2 __attribute__((ext_vector_type(2)));
        char* const o0 = out + (size_t)(c0 * TILE) * so;
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const unsigned vo = vt + lane_row<T, M>(m, lk) * so;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            P2* const o = (P2*)(o0 + (size_t)uniform_row<T, M>(m, j) * so + vo);
#pragma unroll
            for (int h = 0; h < NT / 2; ++h) o[h] = P2{acc.c[m][2 * h][j], acc.c[m][2 * h + 1][j]};
          }
        }
      }
    });
    c0 = c0n;
  }
}

template <typename T>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
void k_sigma_mm(MmParams p) {
  __shared__ __attribute__((aligned(65536))) T buf[mm_lds<T>()];
  mm_unit<T>(p, buf, blockIdx.x & 7, blockIdx.x >> 3);
}

// Grouped launch (serving): the same launch of several products in one grid, on every XCD the phase 2
// units (the long ones) of all products first, then the phase 1 units. A unit does exactly what it does
// in its own product's launch.
struct MmGroup {
  int n, b2[GROUP_MAX + 1], b1[GROUP_MAX + 1];  // first unit of product e on an XCD, by phase
  MmParams e[GROUP_MAX];
};
static_assert(sizeof(MmGroup) <= 4096, "kernel arguments");

template <typename T>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
void k_sigma_mm_group(MmGroup ga) {
  __shared__ __attribute__((aligned(65536))) T buf[mm_lds<T>()];
  int idx = blockIdx.x >> 3, e = 0;
  if (idx < ga.b2[ga.n]) {
    while (idx >= ga.b2[e + 1]) ++e;
    idx -= ga.b2[e];
  } else {
    idx -= ga.b2[ga.n];
    while (idx >= ga.b1[e + 1]) ++e;
    idx += ga.e[e].per2 - ga.b1[e];
  }
  mm_unit<T>(ga.e[e], buf, blockIdx.x & 7, idx);
}

}  // namespace

MmGeometry mm_geometry(const Geometry& g) {
  return MmGeometry{g.nvt, g.nct, g.nvt, g.nct, g.naux, 1};
}
MmGeometry mm_geometry(const AbGeometry& g) {
  return MmGeometry{g.nvta, g.ncta, g.nvtb, g.nctb, g.naux, 0};
}

static SigmaSums sums_of(const MmGeometry& g, Store st, int k, int nsplit) {
  const int64_t zz = (int64_t)g.ncta * g.nctb * TILE * TILE, ld = g.nctb * TILE;
  const MmPlan m = mm_plan(st, g, k, nsplit * k);
  if (m.nslot == 0 || st == Store::BF16) {
    const int ns = m.nslot ? m.nslot : nsplit;
    return {st == Store::F64 ? Store::F64 : Store::F32, ns, zz, k * zz,
            ns, g.nvta * TILE * ld + g.nvtb * TILE, ld, zz, k * zz};
  }
  const int64_t ldo = (g.nctb - g.nvtb) * TILE, zo = (g.ncta - g.nvta) * TILE * ldo;
  return {Store::F64, m.nslot, zz, k * zz, m.nslot * m.ro, m.nslot * k * zz, ldo, zo, k * zo};
}
SigmaSums sigma_sums(const Geometry& g, Store st, int k, int nsplit) {
  return sums_of(mm_geometry(g), st, k, nsplit);
}
SigmaSums sigma_sums(const AbGeometry& g, Store st, int k, int nsplit) {
  return sums_of(mm_geometry(g), st, k, nsplit);
}

// Workspace of the (FP64) sums of k vectors, in matrices of the sigma precision.
static int64_t sum_slots(Store st, const MmGeometry& g, int k, int nslot, int ro) {
  const int64_t zz = (int64_t)g.ncta * g.nctb, zo = (int64_t)(g.ncta - g.nvta) * (g.nctb - g.nvtb);
  if (st == Store::BF16) return (int64_t)nslot * k;  // FP32, both blocks in one matrix
  const int64_t one = (int64_t)nslot * k + ((int64_t)nslot * ro * k * zo + zz - 1) / zz;
  return st == Store::F64 ? one : 2 * one;
}

MmPlan mm_plan(Store st, const MmGeometry& g, int k, int slots) {
  MmPlan m;
  const bool bf = st == Store::BF16;
  if ((bf && (!g.tri || g.nvta < BF_MIN_NVT)) || g.naux < MM_MIN_NAUX || (g.ncta > g.nvta) != (g.nctb > g.nvtb) ||
      g.nvta == 0 || g.nvtb == 0)
    return m;
  const int tiles = k * g.nvtb, wgs = bf ? 256 : 512;  // workgroups the chip holds
  if (tiles < (st == Store::F64 ? MM_MIN_TILES_F64 : (bf ? BF_MIN_TILES : MM_MIN_TILES_F32))) return m;
  const int ota = g.ncta - g.nvta, otb = g.nctb - g.nvtb;
  const int mt = bf ? BF_MT : MT;
  m.npv = (g.nvta + mt - 1) / mt;
  m.npo = (ota + mt - 1) / mt;
  m.items2v = m.npv * ((tiles + MM_BT - 1) / MM_BT);
  m.items2 = m.items2v + m.npo * ((k * otb + MM_BT - 1) / MM_BT);
  // 32-bit lane offsets
  if (!bf && (uint64_t)g.ncta * g.nctb * TILE * TILE * k * 8 * 3 >= (uint64_t(1) << 32)) return m;
  // phase 2 units fill whole rounds of the chip's workgroups as well as they can: the fewest slots
  // within 2 % of the best fill by the virtual block's units
  auto fill = [&](int ns) {
    const int units = m.items2v * ns, rounds = (units + wgs - 1) / wgs;
    return units / (double)(rounds * wgs);
  };
  auto ro_of = [&](int ns) { return bf ? 1 : std::min(MM_RO, g.naux / ns); };
  // (the smallest workspace holds the sums and two buffers of four aux indices a slot, or of one: each
  // number of slots on its own, as fewer slots may take more sums of the occupied block)
  int most = 0, parts = 4;
  auto fits = [&](int ns) {
    return sum_slots(st, g, k, ns, ro_of(ns)) + (bf ? 3 : 2) * (int64_t)parts * ns * k <= slots;
  };
  double best = 0;
  for (;; parts /= 2) {
    most = 0;
    best = 0;
    for (int ns = 1; ns <= std::min(128, g.naux); ++ns)
      if (fits(ns)) {
        most = ns;
        best = std::max(best, fill(ns));
      }
    if (parts == 1 || m.items2v * most >= 0.9 * wgs) break;
  }
  if (most == 0) return m;
  m.nslot = 1;
  while (!fits(m.nslot) || fill(m.nslot) < best - 0.02) ++m.nslot;
  m.ro = ro_of(m.nslot);
  m.qslots = sum_slots(st, g, k, m.nslot, m.ro);
  return m;
}

size_t mm_more(Store st, const MmGeometry& g, int k, int slots) {
  const MmPlan m = mm_plan(st, g, k, slots);
  if (m.nslot == 0) return 0;
  const int64_t len = (g.naux + m.nslot - 1) / m.nslot;
  const int64_t t = std::min<int64_t>(len, 2 * MM_PART) * m.nslot * k * (st == Store::BF16 ? 3 : 2) / 2;
  return (size_t)std::max<int64_t>(0, m.qslots + t - slots);
}

// Longest slot, and the matrices of T that the workspace holds.
static int mm_len(const MmGeometry& g, const MmProduct& a) { return (g.naux + a.m.nslot - 1) / a.m.nslot; }
static int64_t mm_room(const MmProduct& a) { return a.ws_slots - a.m.qslots; }

// Parts of every slot: all of T in one buffer, or as much as two hold.
static int mm_parts(const MmGeometry& g, const MmProduct& a) {
  const int64_t len = mm_len(g, a), room = mm_room(a) / ((int64_t)a.k * a.m.nslot);
  return room >= len ? 1 : (int)((len + room / 2 - 1) / (room / 2));
}

// Whole slots of a launch, half of the workspace, for which a product gives up its parts: those of under
// MM_RUN_PART aux indices each (0: none).
static int mm_whole_slots(const MmGeometry& g, const MmProduct& a) {
  const int len = mm_len(g, a), parts = mm_parts(g, a);
  if (parts == 1 || (len + parts - 1) / parts >= MM_RUN_PART) return 0;
  return (int)(mm_room(a) / 2 / ((int64_t)len * a.k));
}

// Kernel arguments of a product, but for those of one launch (step). slots: those of a launch, whole, or
// 0: all, in parts.
static hipError_t mm_params(Store st, const MmGeometry& g, const MmProduct& a, int slots, MmParams& p) {
  const MmPlan& m = a.m;
  const int k = a.k;
  p = MmParams{};
  p.nvta = g.nvta;
  p.ncta = g.ncta;
  p.nvtb = g.nvtb;
  p.nctb = g.nctb;
  p.nmopa = g.ncta * TILE;
  p.nmopb = g.nctb * TILE;
  p.k = k;
  p.tri = g.tri;
  p.npv = m.npv;
  p.npo = m.npo;
  p.items2v = m.items2v;
  p.items2 = m.items2;
  p.nslot = m.nslot;
  p.ro = m.ro;
  p.naux = g.naux;
  p.La = a.La;
  p.Lb = a.Lb;
  p.UT = a.UT;
  p.ustride = (int64_t)p.nmopb * p.nmopa;
  p.lbstride = (int64_t)p.nmopb * p.nmopb;
  p.qstride = (int64_t)p.nmopa * p.nmopb;
  p.qostride = (int64_t)(g.ncta - g.nvta) * (g.nctb - g.nvtb) * TILE * TILE;
  p.Q = (double*)a.ws;
  p.Qo = p.Q + (int64_t)m.nslot * k * p.qstride;
  const int len = mm_len(g, a);
  const int64_t room = mm_room(a) / ((int64_t)k * m.nslot);
  if (room < 2 && room < len) return hipErrorInvalidValue;
  p.nrun = slots > 0 ? slots : m.nslot;
  p.nparts = slots > 0 ? 1 : mm_parts(g, a);
  p.mc = (len + p.nparts - 1) / p.nparts;
  p.nbs = (p.mc * g.nctb + MM_BT - 1) / MM_BT;
  const int64_t size = st == Store::F64 ? 8 : 4;
  p.T0 = (char*)a.ws + m.qslots * p.qstride * size;
  p.tpart = (int64_t)p.nrun * p.mc * k * p.qstride * size;
  return hipSuccess;
}

// Launch c of a product: phase 2 of part c - 1 (or of run c - 1 of the slots) and phase 1 of part c.
static int mm_launches(const MmParams& p) {
  return (p.nparts > 1 ? p.nparts : (p.nslot + p.nrun - 1) / p.nrun) + 1;
}
static void mm_step(MmParams& p, int c) {
  p.part1 = p.nparts > 1 ? c : 0;
  p.part2 = p.nparts > 1 ? c - 1 : 0;
  p.slot1 = p.nparts > 1 ? 0 : c * p.nrun;
  p.slot2 = p.nparts > 1 ? 0 : (c - 1) * p.nrun;
  p.slots1 = c + 1 < mm_launches(p) ? std::min(p.nrun, p.nslot - p.slot1) : 0;
  p.slots2 = c > 0 ? std::min(p.nrun, p.nslot - p.slot2) : 0;
  p.Tout = p.T0 + (c & 1) * p.tpart;
  p.Tin = p.T0 + ((c + 1) & 1) * p.tpart;
  p.units1 = p.k * p.slots1 * p.nbs;
  p.per1 = (p.units1 + 7) / 8;
  p.per2v = (p.items2v * p.slots2 + 7) / 8;
  p.per2 = p.per2v + ((p.items2 - p.items2v) * p.slots2 * p.ro + 7) / 8;
}

hipError_t launch_sigma_mm(Store st, const MmGeometry& g, const MmProduct& a, hipStream_t s) {
  MmParams p;
  const hipError_t e = mm_params(st, g, a, 0, p);
  if (e != hipSuccess) return e;
  for (int c = 0; c < mm_launches(p); ++c) {
    mm_step(p, c);
    const dim3 grid(8 * (p.per1 + p.per2)), wg(MW * 64);
    if (st == Store::F64)
      hipLaunchKernelGGL(k_sigma_mm<double>, grid, wg, 0, s, p);
    else
      hipLaunchKernelGGL(k_sigma_mm<float>, grid, wg, 0, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_sigma_mm_group(Store st, const MmGeometry* g, const MmProduct* a, int n,
                                 hipStream_t s) {
  if (n < 1 || n > GROUP_MAX) return n == 0 ? hipSuccess : hipErrorInvalidValue;
  if (n == 1) return launch_sigma_mm(st, g[0], a[0], s);
  for (int i = 0; i < n; ++i)
    if (mm_room(a[i]) < std::min(2, mm_len(g[i], a[i])) * (int64_t)a[i].k * a[i].m.nslot)
      return hipErrorInvalidValue;
  // runs of whole slots where they make enough phase 2 units a launch (with the phase 1 units beside them,
  // about as much work). Sigma time of 448 served products at 13/117/457 in FP32, 8 vectors, ms, for at
  // least 256 / 96 / 32 units: 151 / 132 / 133; 512 with 4 vectors, 32 solves in flight 110 / 106 / 108, 4 in
  // flight 113 / 117 / 133.
  int64_t units = 0;
  for (int i = 0; i < n; ++i) units += (int64_t)a[i].m.items2v * mm_whole_slots(g[i], a[i]);
  MmParams p[GROUP_MAX];
  int most = 0;
  for (int i = 0; i < n; ++i) {
    const hipError_t e = mm_params(st, g[i], a[i], units >= 96 ? mm_whole_slots(g[i], a[i]) : 0, p[i]);
    if (e != hipSuccess) return e;
    most = std::max(most, mm_launches(p[i]));
  }
  for (int c = 0; c < most; ++c) {
    MmGroup ga;
    ga.n = 0;
    ga.b2[0] = ga.b1[0] = 0;
    for (int i = 0; i < n; ++i) {
      if (c >= mm_launches(p[i])) continue;
      mm_step(p[i], c);
      ga.b2[ga.n + 1] = ga.b2[ga.n] + p[i].per2;
      ga.b1[ga.n + 1] = ga.b1[ga.n] + p[i].per1;
      ga.e[ga.n++] = p[i];
    }
    const dim3 grid(8 * (ga.b2[ga.n] + ga.b1[ga.n])), wg(MW * 64);
    if (st == Store::F64)
      hipLaunchKernelGGL(k_sigma_mm_group<double>, grid, wg, 0, s, ga);
    else
      hipLaunchKernelGGL(k_sigma_mm_group<float>, grid, wg, 0, s, ga);
  }
  return hipGetLastError();
}

}  // namespace pprpa
