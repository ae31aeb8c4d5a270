// BF16-split sigma contraction as two matrix products (gfx950, restricted blocks): the phases of
// k_sigma_mm.hip on the BF16 matrix cores, operands and T as split planes (sigma_bf16.h).
//
//   phase 1   T[P][kv][col][c] = sum_d U_kv[c][d] L^P[col][d]      (d >= c, c's block)
//   phase 2   Q[kv][r][col]    = sum_{P,c} L^P[r][c] T[P][kv][col][c]   (the two diagonal blocks)
//
// Every operand is rows of contiguous reduction indices, which is what a lane of the MFMA reads (8 of
// one row): U row-major, L^P symmetric, T stored with c contiguous, as FP32 sums split into planes
// (what the one-kernel form splits in registers).
//
// Against the one-kernel form (T in registers, a panel of 4 or 8 column tiles whose L^P rows are
// staged for it alone): a unit of 256 x 128 results stages 24 tiles of 1 KiB a plane for 128 tile
// products, and the columns of all vectors (phase 2) or of all P (phase 1) form one index.
//   * unit: 8 waves, 4 x 4 tiles each (two pairs of row tiles, four column tiles), one unit a CU; 32
//     reduction indices a stage, two LDS buffers for three planes and three for two (144 KB; loads
//     issued in the middle of a stage's products instead of ahead of them, 4-10 % slower);
//   * all planes by tiles of 1 KiB (sigma_bf16.h), whole lines for L2: 101 -> 89 ms at 50/500/1800, six
//     products, against row-major planes;
//   * the two tiles of a pair take its rows in turns of 4, so that a lane's T is 8 consecutive c, 16
//     bytes a plane: whole tiles stored, 89 -> 82 ms (8-byte pieces from two waves before);
//   * a wave's run has its own code for each count of pairs, straight-line within a stage, the next
//     row tile's operands read in the middle of a tile's products (107 -> 101 ms; a switch per stage
//     spills);
//   * the sums of an aux index (an FP32 chain of the c's) are added up in FP32 over the slot: two
//     short chains instead of one of all (P, c), 1.3e-6 -> 3.6e-7 relative error at 50/500/1800 with
//     six products;
//   * launches, slots and parts of T as in k_sigma_mm.hip; phase 1 units in groups of 8 column blocks
//     by 4 vectors, what an XCD reads at a time.
// What bounds it: the loads' latency with one stage (six products) in flight, and T's conversion and
// store in phase 1: with the products cut to a sixth 83 ms of 101 remained, with no loads 69; the
// matrix pipe is busy 60 % of phase 2. Times (us), one-kernel form before -> now: 50/500/1800 six
// products 116573 -> 84000 to 88900 by card (20 vectors; 1.01 to 1.07 PFLOP/s of BF16 products, 3/4 of the
// full contraction's), 40/400/1540 three 26903 -> 20900 to 22300.
#include "internal.h"
#include "sigma_bf16.h"
#include "sigma_mm.h"

namespace pprpa {
namespace {

constexpr int BW = 8;             // waves per workgroup
constexpr int BMT = BF_MT;        // row tiles per panel, 4 a wave
constexpr int BBT = MM_BT;        // column tiles per unit, 4 a wave
constexpr int TB = TILE * KB;     // elements of a staged tile (16 rows x 32)
static_assert(BMT == 2 * BW && BBT == BW, "whole tiles per wave load");

struct BfParams {
  int nvt, nct, nmop, k;
  int npv, npo, evenv, eveno, items2v, items2, nslot, naux;
  int nparts, part1, part2, mc, nbs;
  int units1, per1, per2v, per2;
  const u16* L;
  const u16* U;
  const u16* Tin;
  u16* Tout;
  float* Q;  // [nslot][k][nmop][nmop]
  size_t plane, zplane, tplane;
};

template <int N> struct IntC { static constexpr int v = N; };

template <int NPROD>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void k_sigma_bf16_mm(BfParams p) {
  constexpr int NPL = NPROD == 6 ? 3 : 2;
  constexpr int STAGE = NPL * (BMT + BBT) * TB;  // elements per stage buffer
  constexpr int NBUF = NPL == 3 ? 2 : 3;         // 144 KB
  constexpr int LOADS = 3 * NPL;                 // of a wave, a stage
  __shared__ __attribute__((aligned(1024))) u16 buf[NBUF * STAGE];
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  // pairs of row tiles rg, rg + 4 and column tiles 4 cg .. 4 cg + 3 of the unit (the two waves of a
  // SIMD take different rg, so that the SIMDs share a ragged panel)
  const int rg = w < 4 ? w : 7 - w, cg = w >> 2;
  const int64_t zz = (int64_t)p.nmop * p.nmop;

  // this lane's byte offset in a tile's 16 rows, and of its operand reads
  unsigned va = 64 * (lane >> 2) + 16 * ((lane & 3) ^ swz(lane >> 2));
  // operand reads: the two tiles of a pair take its rows in turns of 4, so that a lane's results of
  // both are 8 consecutive rows (MFMA row 4 lk + j of tile t: row 8 lk + 4 t + j of the pair)
  const int ra = 8 * (li >> 2) + (li & 3);
  const int sa[2] = {ra * KB + 8 * (lk ^ swz(ra)), (ra + 4) * KB + 8 * (lk ^ swz(ra + 4))};
  const int sb = li * KB + 8 * (lk ^ swz(li));
  unsigned cur = 0, put = 0;  // the stage buffers being read and loaded next (elements)
  // direct loads of one stage: row tiles of A from pa on, this wave's column tile of B at pb
  auto issue = [&](const u16* pa, size_t aplane, int mt, const u16* pb, size_t bplane) __attribute__((always_inline)) {
    asm volatile("" : "+v"(va));
    u16* const b = buf + put;
    put = put == (NBUF - 1) * STAGE ? 0 : put + STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = w + BW * h;  // (past a ragged panel its last tile: every stage has LOADS loads)
#pragma unroll
      for (int q = 0; q < NPL; ++q)
        __builtin_amdgcn_global_load_lds(
            (const void*)((const char*)(pa + q * aplane + (size_t)(min(j, mt - 1) * TILE) * p.nmop) + va),
            (lds_ptr_t)(b + (q * BMT + j) * TB), 16, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < NPL; ++q)
      __builtin_amdgcn_global_load_lds((const void*)((const char*)(pb + q * bplane) + va),
                                       (lds_ptr_t)(b + (NPL * BMT + q * BBT + w) * TB), 16, 0, 0);
  };
  // wait for the current stage's loads (this wave's, then everyone's); with three buffers the next
  // stage's, issued after them, stay in flight (more: there is one)
  auto arrive = [&](bool more) __attribute__((always_inline)) {
    constexpr int N = (NBUF - 2) * LOADS;
    if (N > 0 && more)
      __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    else
      __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto advance = [&]() __attribute__((always_inline)) { cur = cur == (NBUF - 1) * STAGE ? 0 : cur + STAGE; };

  f4 acc[4][4];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[s][j] = f4{0, 0, 0, 0};
  };
  // one stage on the first pairs of row tiles of this wave: the next tile's operands are read in the
  // middle of a tile's products
  auto product = [&](auto SC) __attribute__((always_inline)) {
    constexpr int S = 2 * decltype(SC)::v;
    constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {0, 1, 0, 1, 2, 0};
    const u16* const A = buf + cur + 2 * rg * TB;
    const u16* const B = buf + cur + (NPL * BMT + 4 * cg) * TB + sb;
    bf8 bv[4][NPL], av[2][NPL];
#pragma unroll
    for (int q = 0; q < NPL; ++q) av[0][q] = *(const bf8*)(A + sa[0] + q * BMT * TB);
#pragma unroll
    for (int q = 0; q < NPL; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j][q] = *(const bf8*)(B + (q * BBT + j) * TB);
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
      for (int t = 0; t < NPROD; ++t) {
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 < S && t == 1) {
#pragma unroll
          for (int q = 0; q < NPL; ++q)
            av[(s + 1) & 1][q] =
                *(const bf8*)(A + sa[(s + 1) & 1] + (q * BMT + 8 * ((s + 1) >> 1)) * TB);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[s][j] = mfma(av[s & 1][pa[t]], bv[j][pb[t]], acc[s][j]);
      }
    }
  };
  auto pairs_of = [&](int mt) __attribute__((always_inline)) {  // this wave's of mt row tiles
    return max(0, (mt / 2 - rg + 3) >> 2);
  };

  if (idx < p.per2) {
    // ---- phase 2 unit: a slot, a block of columns, a row panel; the virtual block's units first ----
    const bool virt = idx < p.per2v;
    const int items = virt ? p.items2v : p.items2 - p.items2v;
    const int u = virt ? xcd * p.per2v + idx : xcd * (p.per2 - p.per2v) + idx - p.per2v;
    if (u >= items * p.nslot) return;
    const int slot = u / items, it = u - slot * items;
    const int lo = mm_cut(0, p.naux, p.nslot, slot), hi = mm_cut(0, p.naux, p.nslot, slot + 1);
    const int Pa = mm_cut(lo, hi, p.nparts, p.part2), Pb = mm_cut(lo, hi, p.nparts, p.part2 + 1);
    if (Pa >= Pb) return;
    const int npan = virt ? p.npv : p.npo;
    const int nb = it / npan, pan = it - nb * npan;
    const int bt = virt ? p.nvt : p.nct - p.nvt, base = virt ? 0 : p.nvt;
    const bool even = virt ? p.evenv : p.eveno;
    const int t0 = bf_cut(bt, npan, pan, even), mt = bf_cut(bt, npan, pan + 1, even) - t0;
    const int ntot = p.k * bt, kc = p.nct / 2;
    const int jl = min(nb * BBT + w, ntot - 1);  // the column tile this wave loads
    const int jkv = jl / bt, jct = base + jl - jkv * bt;
    const u16* pa = p.L + (size_t)Pa * zz + (size_t)((base + t0) * TILE) * p.nmop;
    const u16* pb = p.Tin + ((size_t)(slot * p.mc) * p.k + jkv) * zz + (size_t)(jct * TILE) * p.nmop;
    const int n = (Pb - Pa) * kc, S = pairs_of(mt);
    int lc = 0;
    auto next = [&]() __attribute__((always_inline)) {
      issue(pa, p.plane, mt, pb, p.tplane);
      pa += TB;
      pb += TB;
      if (++lc == kc) {
        lc = 0;
        pa += zz - kc * TB;
        pb += p.k * zz - kc * TB;
      }
    };
    float* const Q = p.Q + (size_t)slot * p.k * zz + (size_t)((base + t0) * TILE) * p.nmop;
    next();
    if (NBUF > 2 && n > 1) next();
    // (the whole run for each count of pairs: a switch per stage spills registers)
    auto run = [&](auto SC) __attribute__((always_inline)) {
      constexpr int S = 2 * decltype(SC)::v, SS = S > 0 ? S : 1;
      f4 sum[SS][4];
      auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int jo = nb * BBT + 4 * cg + j;
          if (jo < ntot) {  // uniform
            const int kv = jo / bt, ct = base + jo - kv * bt;
            float* const q = Q + (size_t)kv * zz + ct * TILE + li + (size_t)(2 * rg * TILE + 8 * lk) * p.nmop;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                f(q[(size_t)(8 * (s >> 1) * TILE + 4 * (s & 1) + r) * p.nmop], s, j, r);
          }
        }
      };
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[s][j] = f4{0, 0, 0, 0};
      // the sums of a slot go on from one launch to the next
      if (Pa > lo) each([&](float& x, int s, int j, int r) __attribute__((always_inline)) { sum[s][j][r] = x; });
      for (int st = 0; st < n; st += kc) {  // a chain per aux index
        clear();
        for (int c = 0; c < kc; ++c) {
          arrive(st + c + 1 < n);
          if (st + c + NBUF - 1 < n) next();
          product(SC);
          advance();
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int j = 0; j < 4; ++j) sum[s][j] += acc[s][j];
      }
      each([&](float& x, int s, int j, int r) __attribute__((always_inline)) { x = sum[s][j][r]; });
    };
    switch (S) {
      case 2: run(IntC<2>{}); break;
      case 1: run(IntC<1>{}); break;
      default: run(IntC<0>{}); break;
    }
    return;
  }

  // ---- phase 1 unit: one vector, a block of columns of consecutive (P, column tile) ---------------
  const int u = xcd * p.per1 + idx - p.per2;
  if (u >= p.units1) return;
  // (groups of 8 column blocks by up to 4 vectors: what an XCD's units read at a time)
  const int slot = u / (p.k * p.nbs), us = u - slot * p.k * p.nbs;
  const int ng = us / (8 * p.k), nn = min(8, p.nbs - 8 * ng), ug = us - ng * 8 * p.k;
  const int kg = ug / (4 * nn), kn = min(4, p.k - 4 * kg), uk = ug - kg * 4 * nn;
  const int nb = 8 * ng + uk / kn, kv = 4 * kg + uk % kn;
  const int lo = mm_cut(0, p.naux, p.nslot, slot), hi = mm_cut(0, p.naux, p.nslot, slot + 1);
  const int Ppart = mm_cut(lo, hi, p.nparts, p.part1);
  const int ntot = (mm_cut(lo, hi, p.nparts, p.part1 + 1) - Ppart) * p.nct;
  if (nb * BBT >= ntot) return;
  const int jl = min(nb * BBT + w, ntot - 1), jP = jl / p.nct;
  const u16* const pb0 = p.L + (size_t)(Ppart + jP) * zz + (size_t)((jl - jP * p.nct) * TILE) * p.nmop;
  const u16* const pa0 = p.U + (size_t)kv * zz;
  const int npan = p.npv + p.npo;
  // panel i: its first row tile (c), tiles and blocks of 32 of the reduction [b0, b1)
  auto panel = [&](int i, int& c, int& mt, int& b0, int& b1) __attribute__((always_inline)) {
    const bool virt = i < p.npv;
    const int np = virt ? p.npv : p.npo, j = virt ? i : i - p.npv;
    const int bt = virt ? p.nvt : p.nct - p.nvt, base = virt ? 0 : p.nvt;
    const bool even = virt ? p.evenv : p.eveno;
    c = base + bf_cut(bt, np, j, even);
    mt = base + bf_cut(bt, np, j + 1, even) - c;
    b0 = c / 2;
    b1 = (base + bt) / 2;
  };
  int li_ = 0, lc, lmt, lb, lb1;  // the panel and block being loaded, one stage ahead
  panel(0, lc, lmt, lb, lb1);
  auto next = [&]() __attribute__((always_inline)) {
    if (li_ >= npan) return;
    issue(pa0 + (size_t)(lc * TILE) * p.nmop + lb * TB, p.zplane, lmt, pb0 + lb * TB, p.plane);
    if (++lb == lb1 && ++li_ < npan) panel(li_, lc, lmt, lb, lb1);
  };
  next();
  if (NBUF > 2) next();
  for (int i = 0; i < npan; ++i) {
    int c, mt, b0, b1;
    panel(i, c, mt, b0, b1);
    clear();
    int b = b0;
    // the pairs of row tiles that reach the diagonal (c <= d): pair c / 2 + rg + 4 i takes part from
    // that block on
    auto run_to = [&](int end, auto SC) __attribute__((always_inline)) {
      for (; b < end; ++b) {
        arrive(i + 1 < npan || b + 1 < b1);
        next();
        product(SC);
        advance();
      }
    };
    const int mp = mt / 2, f = c / 2 + rg;
    run_to(min(f, b1), IntC<0>{});
    if (mp > rg) run_to(mp > rg + 4 ? min(f + 4, b1) : b1, IntC<1>{});
    if (mp > rg + 4) run_to(b1, IntC<2>{});
    run_to(b1, IntC<0>{});
    const int S = pairs_of(mt);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int jo = nb * BBT + 4 * cg + j;
      if (jo < ntot) {  // uniform
        const int P = jo / p.nct, ct = jo - P * p.nct;
        u16* const o = p.Tout + ((size_t)(slot * p.mc + P) * p.k + kv) * zz +
                       (size_t)(ct * TILE) * p.nmop + bf16_cols(c + 2 * rg) + li * KB + 8 * lk;
#pragma unroll
        for (int s = 0; s < 2; ++s)
          if (s < S) {
            bf8 h[3];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
              __bf16 x, y, z;
              split3(acc[2 * s + (r >> 2)][j][r & 3], x, y, z);
              h[0][r] = x;
              h[1][r] = y;
              h[2][r] = z;
            }
#pragma unroll
            for (int q = 0; q < NPL; ++q) *(bf8*)(o + q * p.tplane + 4 * s * TB) = h[q];
          }
      }
    }
  }
}

}  // namespace

hipError_t launch_sigma_bf16_mm(const MmGeometry& g, const MmPlan& m, int nprod, const void* L,
                                size_t plane, const void* U, size_t zplane, void* ws,
                                int64_t ws_slots, int k, hipStream_t s) {
  const int npl = nprod == 3 ? 2 : 3;
  BfParams p{};
  p.nvt = g.nvta;
  p.nct = g.ncta;
  p.nmop = g.ncta * TILE;
  p.k = k;
  p.npv = m.npv;
  p.npo = m.npo;
  p.evenv = bf_even(g.nvta, m.npv);
  p.eveno = bf_even(g.ncta - g.nvta, m.npo);
  p.items2v = m.items2v;
  p.items2 = m.items2;
  p.nslot = m.nslot;
  p.naux = g.naux;
  p.L = (const u16*)L;
  p.U = (const u16*)U;
  p.Q = (float*)ws;
  p.plane = plane;
  p.zplane = zplane;
  const int64_t zz = (int64_t)p.nmop * p.nmop;
  // parts of T (npl 16-bit planes; the workspace counts FP32 matrices): all of it in one buffer, or
  // as much as two hold
  const int len = (g.naux + m.nslot - 1) / m.nslot;
  const int64_t room = (ws_slots - m.qslots) * 2 / npl / ((int64_t)k * m.nslot);
  if (room < 2 && room < len) return hipErrorInvalidValue;
  p.nparts = room >= len ? 1 : (int)((len + room / 2 - 1) / (room / 2));
  p.mc = (len + p.nparts - 1) / p.nparts;
  p.nbs = (p.mc * g.ncta + BBT - 1) / BBT;
  u16* const t0 = (u16*)((float*)ws + m.qslots * zz);
  p.tplane = (size_t)m.nslot * p.mc * k * zz;
  for (int c = 0; c <= p.nparts; ++c) {  // launch c: phase 2 of part c - 1 and phase 1 of part c
    p.part1 = c;
    p.part2 = c - 1;
    p.Tout = t0 + (c & 1) * npl * p.tplane;
    p.Tin = t0 + ((c + 1) & 1) * npl * p.tplane;
    p.units1 = c < p.nparts ? k * m.nslot * p.nbs : 0;
    p.per1 = (p.units1 + 7) / 8;
    p.per2v = c > 0 ? (m.items2v * m.nslot + 7) / 8 : 0;
    p.per2 = c > 0 ? p.per2v + ((m.items2 - m.items2v) * m.nslot + 7) / 8 : 0;
    const dim3 grid(8 * (p.per1 + p.per2)), wg(BW * 64);
    if (nprod == 3)
      hipLaunchKernelGGL(k_sigma_bf16_mm<3>, grid, wg, 0, s, p);
    else
      hipLaunchKernelGGL(k_sigma_bf16_mm<6>, grid, wg, 0, s, p);
  }
  return hipGetLastError();
}

}  // namespace pprpa
