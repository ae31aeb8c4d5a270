"""GPU: the dense pencil's whole chain (Cholesky, tridiagonal form in one launch, eigenvalues by
Sturm counts, inverse iteration, back-transformation) at the orders where its kernels change:
97 (the first order on many workgroups), 256 / 258 and 511 / 513 (columns a lane and rows a wave of
the reduction), 1087 / 1089 (its widest rows, v kept in registers or read again), 2046 / 2052 (the
reduction in one launch or two launches a step, the vectors in LDS and registers or in memory), against
the oracle's whole spectrum.

The NTO weights of random vectors, which take the same reduction for several matrices at once, at
block orders 2 / 3 (one workgroup or several), around the product kernel's tiles of 32, 256 / 257,
and with more matrices than one launch holds (64 of order 130: 5 workgroups each).

Tolerances as in the other tests of these calls: roots and residuals 1e-9, W-norms 1e-10, energies
1e-10 Ha up to n = 513 and 1e-9 Ha above; NTO weights and densities 1e-12 of the largest.
"""
import sys

import numpy as np
import pytest

from oracle import pprpa_oracle as O
from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nocc,nvir,n", [(3, 13, 97), (2, 22, 256), (14, 17, 258), (14, 28, 511),
                                         (12, 29, 513), (3, 46, 1087), (32, 33, 1089),
                                         (23, 59, 2046), (8, 63, 2052)])
def test_dense_chain_at_the_kernels_edges(nocc, nvir, n):
    print("dense chain", n, flush=True)
    sys.stdout.flush()
    eps = gen.orbital_energies(61, nocc, nvir)
    L = gen.lpq_full(61, nocc + nvir, 60)
    sp = O.active_space(eps, L, nocc)
    A, B, C = O.build_matrices(sp, "singlet")
    om, _, sg = O.solve_definite(O.pprpa_matrix(A, B, C), A.shape[0], O.midgap(sp))
    ec, _ = O.correlation_energy(om[sg > 0], om[sg < 0], A, C)
    with P.PpRPA(eps, L, nocc, mult="singlet", dense=True) as ctx:
        assert ctx.n == n
        M = ctx.dense_matrix()
        w = np.r_[np.ones(ctx.n_pp), -np.ones(ctx.n_hh)]
        for channel, ref in (("pp", np.sort(om[sg > 0])), ("hh", np.sort(om[sg < 0])[::-1])):
            k = min(5, len(ref))
            r = ctx.davidson(k, direct=True, vectors=True, channel=channel)
            assert np.max(np.abs(r["omega"] - ref[:k])) <= 1e-9
            Z = r["vecs"]
            assert np.max(np.abs(M @ Z.T - (w[:, None] * Z.T) * r["omega"][None, :])) <= 1e-9
            assert np.allclose(np.einsum("ij,j,ij->i", Z, w, Z), 1.0 if channel == "pp" else -1.0,
                               atol=1e-10)
        e = ctx.correlation_energy()
    assert abs(e["ec_pp"] - ec) <= (1e-10 if n <= 513 else 1e-9)
    assert abs(e["ec_hh"] - ec) <= (1e-10 if n <= 513 else 1e-9)


@pytest.mark.parametrize("nocc,nvir,k", [(2, 3, 3), (3, 33, 5), (31, 32, 2), (33, 256, 2),
                                         (1, 257, 3), (4, 130, 64)])
def test_nto_weights_at_the_kernels_edges(nocc, nvir, k):
    print("nto", nocc, nvir, k, flush=True)
    sys.stdout.flush()
    eps, L = gen.orbital_energies(62, nocc, nvir), gen.lpq_full(62, nocc + nvir, 8)
    with P.PpRPA(eps, L, nocc, mult="singlet") as ctx:
        Z = gen.random_vectors(63, k, ctx.n)
        res = ctx.nto(Z)
    for j, z in enumerate(Z):
        lp, lh, _ = O.nto(z, nvir, nocc, "singlet")
        Dv, Do = O.density_2e(z, nvir, nocc, "singlet")
        for got, ref in ((res["lam_p"], lp), (res["lam_h"], lh), (res["d_vv"], Dv), (res["d_oo"], Do)):
            assert np.max(np.abs(got[j] - ref)) <= 1e-12 * max(np.abs(ref).max(), 1e-300)
