"""Dense solves beside another stream's sigma products, which hold the compute units: the workgroups of
the one-launch tridiagonal reduction (k_tridiag.hip) then start one by one as units come free. The
direct solve with vectors (the reduction that keeps its reflections), the correlation energy and the NTO
weights give the same bits as alone."""
import threading

import numpy as np
import pytest

from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu


def busy_products(stop, errors):
    """Blocks of 20 vectors, one product after the other, each filling the chip for milliseconds."""
    try:
        import torch
        nocc, nvir, naux = 20, 200, 700
        idx = np.arange(nocc + nvir)
        dev = torch.device("cuda:0")
        L = gen.lpq_block_torch(5, nocc + nvir, naux, idx, idx, np.arange(naux), dev)
        eps = torch.from_numpy(gen.orbital_energies(5, nocc, nvir)).to(dev)
        torch.cuda.synchronize()
        with P.PpRPA(eps, L, nocc) as ctx:
            z = torch.from_numpy(gen.random_vectors(3, 20, ctx.n)).to(dev)
            out = torch.empty_like(z)
            torch.cuda.synchronize()
            for _ in range(2000):
                if stop.is_set():
                    break
                ctx.matvec(z, out=out)
    except Exception as e:  # reported by the test
        errors.append(e)


@pytest.mark.parametrize("nocc,nvir,repeats", [(5, 20, 20), (8, 45, 6)])
def test_dense_solves_beside_sigma_products(nocc, nvir, repeats):
    eps, L = gen.orbital_energies(71, nocc, nvir), gen.lpq_full(71, nocc + nvir, 60)
    with P.PpRPA(eps, L, nocc, mult="singlet", dense=True) as ctx:
        z = gen.random_vectors(72, 4, ctx.n)

        def solve():
            r = ctx.davidson(5, direct=True, vectors=True)
            return [r["omega"], r["vecs"], np.array(list(ctx.correlation_energy().values())), ctx.nto(z)["lam_p"]]

        alone = solve()
        stop, errors = threading.Event(), []
        t = threading.Thread(target=busy_products, args=(stop, errors))
        t.start()
        try:
            for i in range(repeats):
                print("dense beside sigma", nocc, nvir, i, flush=True)
                for got, ref in zip(solve(), alone):
                    assert np.array_equal(got, ref), i
        finally:
            stop.set()
            t.join()
        assert not errors, errors
