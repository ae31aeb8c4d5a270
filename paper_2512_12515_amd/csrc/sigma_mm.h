// The two-product sigma contraction (k_sigma_mm.hip): geometry, plan and kernel arguments.
#pragma once

#include <algorithm>

#include "internal.h"

namespace pprpa {

constexpr int MM_MT = 8;      // row tiles per panel
constexpr int MM_BT = 8;      // column tiles per unit
constexpr int BF_MT = 16;     // row tiles per panel of the BF16 form
// Aux indices of a part below which a product in a group takes runs of whole slots instead (requests/s served,
// parts -> runs: 13/117/457 FP64, 7 vectors, parts of one 226 -> 254; 15/150/550 FP32, 5 vectors, parts of two
// 244 -> 256, FP64, 8 vectors, parts of four 126.7 -> 126.6; 20/200/700 FP64, 5 vectors, parts of four
// 59.6 -> 56.6).
constexpr int MM_RUN_PART = 4;
constexpr int MM_RO = 8;      // most slots of the occupied block per slot of the virtual one
// Fewest column tiles of a block of vectors (k x virtual tiles) from which this form runs. us, the
// one-kernel form -> this one: FP64 5/20/100 8 vectors (16 tiles) 66 -> 57, 13/117/457 1 vector (8)
// 178 -> 226, 20/200/700 1 vector (13) 735 -> 696; FP32 5/20/100 8 vectors (16) 64 -> 85,
// 8/80/300 4 vectors (20) 143 -> 98.
constexpr int MM_MIN_TILES_F64 = 16;
constexpr int MM_MIN_TILES_F32 = 18;
// BF16: fewest column tiles and virtual tiles. us, the one-kernel form -> this one, six / three products:
// 20/200/700 20 vectors (280 tiles) 4543 -> 4126 / 3060 -> 2737, 10 (140) 2302 -> 2361 / 1586 -> 1438;
// 20/288/300 20 (360) 4160 -> 3630 / 2658 -> 2150; 40/400/1540 12 (312) 33.2e3 -> 29.9e3 / 20.1e3 -> 16.5e3,
// 2 (52) 5702 -> 5547 / 3426 -> 3658; 50/500/1800 20 (640) 117e3 -> 86e3 / 65.8e3 -> 46.3e3; 13/117/457 20
// (8 virtual tiles) 814 -> 1092 / 636 -> 722.
constexpr int BF_MIN_TILES = 160;
constexpr int BF_MIN_NVT = 13;
// Fewest aux indices: below, the one-kernel form has a split for every aux index whatever the block
// width, and a vector's sigma does not depend on the block around it; that stays so.
constexpr int MM_MIN_NAUX = 96;
// Workspace that a context outside a slab takes at most. FP64 products with the least / 1 GB / 1536 MB /
// 4 GB, us: 20/200/700, 20 vectors 8435 / 8293 / 7881 / 7740, 10 vectors 4364 / 4251 / 4100 / 3964;
// 13/117/457, 7 vectors 685 / 546 / 561 / 547. hipMalloc and hipFree of one buffer take 24 us up to 64 MB, 0.3 ms up to 1536 MB,
// 0.57 ms at 2 GB and 90 to 120 ms from 3 GB on (some hipMallocs after such a hipFree as long), and a
// build with its release 0.87 ms (13/117/457) and 1.1 ms (20/200/700) up to 1536 MB, 1.2 and 1.4 ms with 4 GB.
// Contexts of 32 vectors whose least is under MM_WORKSPACE_MIN stay under it: at 5/20/100 (56 MB) 20 vectors
// take 62 us either way, and the build half of the 0.5 ms. Narrower ones, whose blocks are as wide as the
// least is made for, do not: 10/60/220, 4 vectors of 4 120 -> 87 us (the one-kernel form 100).
constexpr size_t MM_WORKSPACE = size_t(1536) << 20;
constexpr size_t MM_WORKSPACE_MIN = size_t(64) << 20;
// What all contexts of the process take beyond their least on a device, and the share of the device's free
// memory that one takes in all: a program with many contexts, or with little memory left, keeps nearly
// all of it for its own.
constexpr size_t MM_WORKSPACE_MORE = size_t(8) << 30;
constexpr size_t MM_WORKSPACE_SHARE = 16;

// Alpha (rows, c) and beta (d, columns) tiles, virtual block first; a restricted context has both
// alike and takes the upper triangle of U (tri).
struct MmGeometry {
  int nvta = 0, ncta = 0, nvtb = 0, nctb = 0, naux = 0, tri = 0;
};

// Decomposition of one product of k vectors, a function of its sizes alone (its sums do not depend
// on the workspace): slots, each a contiguous share of the aux index with its own sums (the
// occupied block's short units take ro-ths of them), row panels per block and phase 2 work items
// (row panel, column block). nslot = 0: the smallest workspace a context may have does not hold
// this form.
struct MmPlan {
  int nslot = 0, ro = 1, npv = 0, npo = 0, items2v = 0, items2 = 0;
  int64_t qslots = 0;  // workspace of the sums, in matrices of the sigma precision
};
// First element of piece i of n of [lo, hi).
__host__ __device__ inline int mm_cut(int lo, int hi, int n, int i) {
  return lo + (int)((int64_t)(hi - lo) * i / n);
}

// First row tile of panel i of n of bt tiles, BF16: even shares of the pairs of tiles, or of their rows
// of four (a pair for each of four waves), whose last one is as it comes.
__host__ __device__ inline int bf_cut(int bt, int n, int i, bool even) {
  const int cut = even ? bt / 2 * i / n * 2 : (bt + 7) / 8 * i / n * 8;
  return cut < bt ? cut : bt;
}
// Even shares as long as they make no more rows (26 tiles as 14 + 12 rather than 16 + 10: 40/400/1540
// 5 % faster; but 24 as 16 + 8, 3 rows).
inline bool bf_even(int bt, int n) {
  int rows = 0;
  for (int i = 0; i < n; ++i) rows += (bf_cut(bt, n, i + 1, true) - bf_cut(bt, n, i, true) + 7) / 8;
  return rows == (bt + 7) / 8;
}

struct MmParams {
  int nvta, ncta, nvtb, nctb, nmopa, nmopb, k, tri;
  int npv, npo, items2v, items2, nslot, ro, naux;
  int nparts, part1, part2;  // parts of every slot's aux indices: this launch's phase 1 and phase 2
  int nrun, slot1, slots1, slot2, slots2;  // slots of a launch, at most; this one's first and number
  int mc, nbs;               // most aux indices of a slot's part, their column blocks
  int units1, per1, per2v, per2;
  const void* La;    // [naux][nmopa][nmopa]
  const void* Lb;    // [naux][nmopb][nmopb]
  const void* UT;    // [k][nmopb][nmopa]
  const void* Tin;   // [slots2][mc][nmopa][k][nmopb]
  void* Tout;
  char* T0;          // the buffers of T, tpart bytes each
  int64_t tpart;
  double* Q;         // [nslot][k][nmopa][nmopb], the virtual block
  double* Qo;        // [nslot ro][k][nopa][nopb], the occupied block
  int64_t ustride, lbstride, qstride, qostride;
};

// Workspace beyond `slots` matrices that a product of k vectors uses to advantage, in matrices: that of
// parts of MM_PART aux indices. A served request gets it while the arena is mostly free (requests/s, least -> more
// workspace, the one-kernel form in brackets; 13/117/457, 4 roots, 32 solves in flight: FP64 322 -> 345 (311),
// FP32 389 -> 457 (403); 4 in flight: 239 -> 277 (254), 289 -> 347 (318)).
constexpr int MM_PART = 8;
size_t mm_more(Store st, const MmGeometry& g, int k, int slots);

MmGeometry mm_geometry(const Geometry& g);
MmGeometry mm_geometry(const AbGeometry& g);
// slots: the smallest workspace in units of one nmopa x nmopb matrix of the sigma precision.
MmPlan mm_plan(Store st, const MmGeometry& g, int k, int slots);
// One product of k vectors. ws: Q, Qo, then T, ws_slots units (at least the plan's slots).
struct MmProduct {
  MmPlan m;
  const void *La, *Lb, *UT;
  void* ws;
  int64_t ws_slots;
  int k;
};
hipError_t launch_sigma_mm(Store st, const MmGeometry& g, const MmProduct& a, hipStream_t s);
// Up to GROUP_MAX products of one precision side by side, each bit for bit as by itself.
hipError_t launch_sigma_mm_group(Store st, const MmGeometry* g, const MmProduct* a, int n,
                                 hipStream_t s);
// One product for BF16 planes of L (plane elements apart) and U (row-major, zplane apart), restricted.
hipError_t launch_sigma_bf16_mm(const MmGeometry& g, const MmPlan& m, int nprod, const void* L,
                                size_t plane, const void* U, size_t zplane, void* ws,
                                int64_t ws_slots, int k, hipStream_t s);

}  // namespace pprpa
