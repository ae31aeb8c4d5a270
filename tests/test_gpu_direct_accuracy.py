"""The roots of the direct solve to the rounding of the reduction: against the Rayleigh quotients of their
own vectors in extended precision, whose error is of second order in the vectors'. The pencil's tridiagonal
form has a norm of about 10 here; 4 roundings of it are allowed, 9e-15 (with the last bracket of the
multisection kept as it was before counts out of order, one root in two hundred was off by up to 2e-14)."""
import numpy as np
import pytest

from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mult", ["singlet", "triplet"])
def test_direct_roots(mult):
    nocc, nvir, naux = 5, 20, 100
    worst = 0.0
    for seed in range(24):
        eps, L = gen.orbital_energies(seed, nocc, nvir), gen.lpq_full(seed, nocc + nvir, naux)
        with P.PpRPA(eps, L, nocc, mult=mult, dense=True) as ctx:
            M = ctx.dense_matrix().astype(np.longdouble)
            w = np.r_[np.ones(ctx.n_pp), -np.ones(ctx.n_hh)].astype(np.longdouble)
            for channel in ("pp", "hh"):
                r = ctx.davidson(10, direct=True, vectors=True, channel=channel)
                Z = r["vecs"].astype(np.longdouble)
                ref = np.einsum("ij,ij->i", Z @ M, Z) / np.einsum("ij,j,ij->i", Z, w, Z)
                worst = max(worst, float(np.max(np.abs(r["omega"] - ref))))
    print("direct roots", mult, worst, flush=True)
    assert worst <= 9e-15
