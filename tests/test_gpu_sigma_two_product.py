"""Sigma as two matrix products (k_sigma_mm.hip) against the oracle's factorised sigma, at the sizes
where its decomposition changes: the block widths on both sides of its threshold, every number of row
tiles in a panel (1 to 8 and the two-panel splits of 9 and 13), column blocks with a ragged end,
occupied blocks of one and two panels' tiles, aux counts at the threshold and beyond, and
a served context, whose small workspace takes the product in many parts, against its own context.

Tolerances: FP64 1e-12 of max|M z| (sums of at most 1e5 terms of relative rounding 1.1e-16, with two
orders of margin for their growth); FP32 2e-6 (FP32 rounding 6e-8 over chains of at most 4096 terms
folded into FP64, times sqrt(4096 / 4) for the random walk of a four-term step)."""
import numpy as np
import pytest

from oracle import pprpa_oracle as O
from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 2e-6}


def check(nocc, nvir, naux, mult, prec, ks, seed=7):
    print("two-product sigma", nocc, nvir, naux, mult, prec, ks, flush=True)
    eps = gen.orbital_energies(seed, nocc, nvir)
    L = gen.lpq_full(seed, nocc + nvir, naux)
    sp = O.active_space(eps, L, nocc)
    with P.PpRPA(eps, L, nocc, mult=mult, prec=prec) as ctx:
        for k in ks:
            z = gen.random_vectors(3 + k, k, ctx.n)
            ref = np.stack([O.sigma_factorised(sp, mult, v) for v in z])
            assert np.max(np.abs(ctx.matvec(z) - ref)) <= TOL[prec] * np.abs(ref).max(), k


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nocc,nvir,naux,ks", [
    (4, 16, 102, (15, 16, 17, 18, 32)),    # one tile: the two thresholds
    (3, 31, 99, (7, 8, 9, 20)),            # 2
    (17, 40, 97, (5, 6, 7)),               # 3; two occupied tiles
    (2, 64, 98, (4, 5)),                   # 4
    (5, 73, 101, (4, 8)),                  # 5
    (35, 90, 96, (2, 3, 4)),               # 6; three occupied tiles
    (4, 112, 100, (3,)),                    # 7
    (6, 121, 96, (3, 5)),                  # 8
    (1, 135, 97, (2, 7)),                  # 9 = 4 + 5
])
def test_panels_and_thresholds(prec, nocc, nvir, naux, ks):
    for mult in ("singlet", "triplet"):
        check(nocc, nvir, naux, mult, prec, ks)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("naux", [95, 96, 129, 300])
def test_aux_counts(prec, naux):
    check(9, 50, naux, "singlet", prec, (5, 16, 32))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_served_equals_standalone(prec):
    """A served request's workspace holds T in parts, a standalone context's in one: the same bits."""
    import torch
    nocc, nvir, naux = 20, 200, 380
    eps = gen.orbital_energies(5, nocc, nvir)
    idx = np.arange(nocc + nvir)
    dev = torch.device("cuda:0")
    L = 0.7 * gen.lpq_block_torch(5, nocc + nvir, naux, idx, idx, np.arange(naux), dev)
    eps = torch.from_numpy(eps).to(dev)
    torch.cuda.synchronize()
    print("two-product sigma served", prec, flush=True)
    with P.PpRPA(eps, L, nocc, mult="triplet", prec=prec) as ctx:
        own = ctx.davidson(10, tol=1e-5)["omega"]
    with P.Server(4 << 30, 2) as srv:
        r = srv.wait(srv.submit(eps, L, nocc, 10, mult="triplet", prec=prec, tol=1e-5), timeout=120.0)
    assert r["status"] == P.binding.OK, r["message"]
    assert np.array_equal(r["omega"], own)


@pytest.mark.parametrize("nocc,nvir,naux,nroot,prec", [(59, 30, 96, 24, "fp64"), (50, 20, 130, 16, "fp64"),
                                                       (44, 49, 173, 14, "fp32")])
def test_served_with_a_large_occupied_block(nocc, nvir, naux, nroot, prec):
    """Occupied blocks as large as the virtual one, where fewer slots take more sums: the smallest
    workspace has to hold the number of slots that is taken, not only a larger one."""
    print("two-product sigma served, large occupied block", nocc, nvir, naux, nroot, prec, flush=True)
    eps = gen.orbital_energies(9, nocc, nvir)
    L = 0.7 * gen.lpq_full(9, nocc + nvir, naux)
    with P.PpRPA(eps, L, nocc, mult="singlet", prec=prec) as ctx:
        own = ctx.davidson(nroot, block=nroot, tol=1e-4)["omega"]
    with P.Server(2 << 30, 2) as srv:
        r = srv.wait(srv.submit(eps, L, nocc, nroot, mult="singlet", prec=prec, block=nroot, tol=1e-4),
                     timeout=60.0)
    assert r["status"] == P.binding.OK, r["message"]
    assert np.array_equal(r["omega"], own)
