// The two-product sigma contraction (k_sigma_mm.hip): geometry, plan and kernel arguments.
#pragma once

#include <algorithm>

#include "internal.h"

namespace pprpa {

constexpr int MM_MT = 8;      // row tiles per panel
constexpr int MM_BT = 8;      // column tiles per unit
constexpr int MM_RO = 8;      // most slots of the occupied block per slot of the virtual one
// Fewest column tiles of a block of vectors (k x virtual tiles) from which this form runs. us, the
// one-kernel form -> this one: FP64 5/20/100 8 vectors (16 tiles) 66 -> 57, 13/117/457 1 vector (8)
// 178 -> 226, 20/200/700 1 vector (13) 735 -> 696; FP32 5/20/100 8 vectors (16) 64 -> 85,
// 8/80/300 4 vectors (20) 143 -> 98.
constexpr int MM_MIN_TILES_F64 = 16;
constexpr int MM_MIN_TILES_F32 = 18;
// Fewest aux indices: below, the one-kernel form has a split for every aux index whatever the block
// width, and a vector's sigma does not depend on the block around it; that stays so.
constexpr int MM_MIN_NAUX = 96;
// Workspace that a context outside a slab takes at most (20/200/700, 20 vectors: 8610 us with the
// least workspace, 7902 with 2 GB, 7679 with 4 GB, 8097 with 8 GB, where the phases no longer share
// launches).
constexpr size_t MM_WORKSPACE = size_t(4) << 30;

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

struct MmParams {
  int nvta, ncta, nvtb, nctb, nmopa, nmopb, k, tri;
  int npv, npo, items2v, items2, nslot, ro, naux;
  int nparts, part1, part2;  // parts of every slot's aux indices: this launch's phase 1 and phase 2
  int mc, nbs;               // most aux indices of a slot's part, their column blocks
  int units1, per1, per2v, per2;
  const void* La;    // [naux][nmopa][nmopa]
  const void* Lb;    // [naux][nmopb][nmopb]
  const void* UT;    // [k][nmopb][nmopa]
  const void* Tin;   // [nslot][mc][nmopa][k][nmopb]
  void* Tout;
  double* Q;         // [nslot][k][nmopa][nmopb], the virtual block
  double* Qo;        // [nslot ro][k][nopa][nopb], the occupied block
  int64_t ustride, lbstride, qstride, qostride;
};

MmGeometry mm_geometry(const Geometry& g);
MmGeometry mm_geometry(const AbGeometry& g);
// slots: the smallest workspace in units of one nmopa x nmopb matrix of the sigma precision.
MmPlan mm_plan(Store st, const MmGeometry& g, int k, int slots);
// ws: Q, Qo, then T, ws_slots units (at least the plan's slots).
hipError_t launch_sigma_mm(Store st, const MmGeometry& g, const MmPlan& m, const void* La,
                           const void* Lb, const void* UT, void* ws, int64_t ws_slots, int k,
                           hipStream_t s);

}  // namespace pprpa
