"""GPU: the dense pencil's whole chain (Cholesky, tridiagonal form in one launch, eigenvalues by
Sturm counts, inverse iteration, back-transformation) at the orders where its kernels change:
97 (the first order on many workgroups), 256 / 258 and 511 / 513 (columns a lane and rows a wave of
the reduction), 1087 / 1089 (the reduction in one launch or two launches a step), 2046 / 2052 (the
vectors in LDS and registers or in memory), against the oracle's whole spectrum.

Tolerances as in the other tests of these calls: roots and residuals 1e-9, W-norms 1e-10, energies
1e-10 Ha up to n = 513 and 1e-9 Ha above.
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
