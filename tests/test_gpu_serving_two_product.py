"""Served requests whose sigma runs as two matrix products side by side in one grid (k_sigma_mm.hip),
in parts of the aux index or in runs of whole slots, and beside requests of the other kernels: every
result is bit for bit that of the request's own context."""
import numpy as np
import pytest

from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("sizes,count,slots", [
    ([(13, 117, 457, 5)], 20, 20),                      # 8 tiles, 5 vectors: runs of slots; two grids
    ([(13, 117, 457, 5)], 2, 2),                        # too few for runs: parts of one aux index
    ([(5, 31, 100, 10), (7, 70, 120, 8), (20, 130, 200, 6), (3, 15, 97, 18), (4, 20, 60, 4)], 30, 30),
    ([(40, 60, 150, 12), (2, 200, 300, 9)], 10, 10),    # large occupied blocks; 13 tiles
])
def test_each_as_by_itself(prec, sizes, count, slots):
    problems, own = [], []
    for i, (nocc, nvir, naux, nroot) in enumerate(sizes):
        eps, L = gen.orbital_energies(90 + i, nocc, nvir), 0.3 * gen.lpq_full(90 + i, nocc + nvir, naux)
        problems.append((eps, L, nocc, nroot))
        with P.PpRPA(eps, L, nocc, prec=prec) as ctx:
            own.append(ctx.davidson(nroot, block=nroot, tol=1e-4)["omega"])
    print("served two-product", prec, sizes, count, flush=True)
    with P.Server(24 << 30, slots) as srv:
        tickets = []
        for i in range(count):
            eps, L, nocc, nroot = problems[i % len(problems)]
            tickets.append(srv.submit(eps, L, nocc, nroot, prec=prec, block=nroot, tol=1e-4))
        for i, t in enumerate(tickets):
            r = srv.wait(t, timeout=60.0)
            assert r["status"] == P.binding.OK, r["message"]
            assert np.array_equal(r["omega"], own[i % len(problems)]), i


def test_more_workspace_while_the_arena_is_free():
    """A request has the same result with the workspace of a roomy arena, of one that has room for the
    least only, and among many, of which the first have more; the arena's account ends at zero."""
    nocc, nvir, naux, nroot = 13, 117, 457, 5
    eps, L = gen.orbital_energies(97, nocc, nvir), 0.3 * gen.lpq_full(97, nocc + nvir, naux)
    with P.PpRPA(eps, L, nocc) as ctx:
        own = ctx.davidson(nroot, block=nroot, tol=1e-4)["omega"]
    held = {}
    footprint = 0
    for name, budget, count, slots in (("roomy", 16 << 30, 1, 1), ("least", None, 1, 1), ("many", None, 12, 12)):
        budget = budget or (footprint + (1 << 20) if name == "least" else 16 * footprint)
        print("served workspace", name, budget, flush=True)
        with P.Server(budget, slots) as srv:
            tickets = [srv.submit(eps, L, nocc, nroot, block=nroot, tol=1e-4) for _ in range(count)]
            for t in tickets:
                r = srv.wait(t, timeout=60.0)
                assert r["status"] == P.binding.OK, r["message"]
                assert np.array_equal(r["omega"], own)
                footprint = r["footprint"]
            st = srv.stats()
        assert st["reserved"] == 0 and st["peak_reserved"] <= budget
        held[name] = st["peak_reserved"]
    assert held["least"] == footprint and held["roomy"] > footprint
    assert held["many"] <= 12 * footprint + 16 * footprint // 4
