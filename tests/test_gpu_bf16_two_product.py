"""BF16 sigma as two matrix products (k_sigma_bf16_mm.hip) against the oracle's factorised sigma, at
the sizes where its decomposition changes: block widths on both sides of its threshold of 160 column
tiles, row panels of one and two rows of pairs with full and ragged ends (7, 8, 10, 13 and 17 pairs of
row tiles), ragged column blocks, occupied blocks of one and several pairs, aux counts at its threshold,
and a served context, whose small workspace takes the product in parts, against its own context.

Tolerances, of max|M z|: six products 4e-6 (planes of 24 bits, 1.2e-7, and FP32 sums of up to 600
terms a chain: 6e-8 sqrt(600) = 1.5e-6, with a margin for the largest element), three products 2e-5
(the dropped mid-mid term 2^-16 = 1.5e-5 of a single product, falling with the sum)."""
import numpy as np
import pytest

from oracle import pprpa_oracle as O
from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu

TOL = {"bf16x6": 4e-6, "bf16x3": 2e-5}


@pytest.mark.parametrize("prec", ["bf16x6", "bf16x3"])
@pytest.mark.parametrize("nocc,nvir,naux,ks", [
    (4, 193, 97, (11, 12, 13)),     # 7 pairs: 154, 168, 182 column tiles
    (33, 256, 96, (9, 10, 11)),     # 8 pairs; two occupied pairs
    (1, 310, 101, (7, 8, 9)),       # 10 = 4 + 6
    (70, 401, 99, (6, 7)),          # 13 = 8 + 5; three occupied pairs
    (5, 513, 96, (5,)),             # 17 = 4 + 8 + 5
    (20, 210, 95, (20,)), (20, 210, 130, (31,)),
])
def test_panels_and_thresholds(prec, nocc, nvir, naux, ks):
    for mult in ("singlet", "triplet"):
        print("bf16 two-product sigma", nocc, nvir, naux, mult, prec, ks, flush=True)
        eps = gen.orbital_energies(8, nocc, nvir)
        L = gen.lpq_full(8, nocc + nvir, naux)
        sp = O.active_space(eps, L, nocc)
        with P.PpRPA(eps, L, nocc, mult=mult, prec=prec) as ctx:
            for k in ks:
                z = gen.random_vectors(3 + k, k, ctx.n)
                out = ctx.matvec(z)
                for j in sorted({0, k // 2, k - 1}):
                    ref = O.sigma_factorised(sp, mult, z[j])
                    assert np.max(np.abs(out[j] - ref)) <= TOL[prec] * np.abs(ref).max(), (k, j)


@pytest.mark.parametrize("prec", ["bf16x6", "bf16x3"])
def test_served_equals_standalone(prec):
    """A served request's workspace holds T in parts, a standalone context's in fewer: the same bits."""
    import torch
    nocc, nvir, naux = 20, 200, 380
    eps = gen.orbital_energies(5, nocc, nvir)
    idx = np.arange(nocc + nvir)
    dev = torch.device("cuda:0")
    L = 0.7 * gen.lpq_block_torch(5, nocc + nvir, naux, idx, idx, np.arange(naux), dev)
    eps = torch.from_numpy(eps).to(dev)
    torch.cuda.synchronize()
    print("bf16 two-product sigma served", prec, flush=True)
    with P.PpRPA(eps, L, nocc, mult="triplet", prec=prec) as ctx:
        own = ctx.davidson(16, tol=1e-3)["omega"]
    with P.Server(4 << 30, 2) as srv:
        r = srv.wait(srv.submit(eps, L, nocc, 16, mult="triplet", prec=prec, tol=1e-3), timeout=60.0)
    assert r["status"] == P.binding.OK, r["message"]
    assert np.array_equal(r["omega"], own)
