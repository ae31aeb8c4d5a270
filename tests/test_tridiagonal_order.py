"""The order of reads and stores in the one-launch tridiagonal reduction (k_tridiag.hip) when its
workgroups start at different times, in a NumPy model of the kernel's data flow: G workgroups own the
rows cyclically, read row 0 and their rows when they start, exchange p and row k + 1 once a step through
slots that are written once, and the owner of row k stores the reflection into row k of S.

Workgroups start when compute units come free, in any order and, beside another stream's kernels, at any
time. The results may not depend on it: they are the same bits for every workgroup in turn starting only
when all others wait for it. Stored ahead of the exchange (the owner of row 0 before it has heard of any
other workgroup), reflection 0 reaches a late workgroup as its row 0; the model shows that too, so that
it is known to see such a fault."""
import numpy as np
import pytest


def workgroup(g, G, S, slots, out, store_early):
    """One workgroup; yields while a slot that it polls is empty."""
    n = len(S)
    rows = list(range(g, n, G))
    A = {r: S[r].copy() for r in rows}
    x = S[0].copy()
    x[0] = 0.0
    for k in range(n - 2):
        x0, nrm = x[k + 1], np.sqrt(x[k + 1:] @ x[k + 1:])
        alpha = -nrm if x0 > 0.0 else nrm
        v = np.where(np.arange(n) > k, x, 0.0)
        v[k + 1] = x0 - alpha
        beta = 1.0 / (nrm * nrm + abs(x0) * nrm)

        def keep():
            if k in A:
                S[k, k + 1:] = v[k + 1:]
                out["beta"][k] = beta

        if store_early:
            keep()
        if k + 1 in A:
            slots[k, "row"] = A[k + 1].copy()
        for r in rows:
            if r > k:
                slots[k, r] = beta * (A[r] @ v)
        while (k, "row") not in slots or any((k, r) not in slots for r in range(k + 1, n)):
            yield
        p, row = np.array([slots.get((k, r), 0.0) for r in range(n)]), slots[k, "row"]
        w = p - 0.5 * beta * (p @ v) * v
        x = row - (v[k + 1] * w + w[k + 1] * v)
        if g == 0:
            out["e"][k], out["d"][k + 1] = alpha, x[k + 1]
        for r in rows:
            if r > k:
                A[r] = A[r] - (v[r] * w + w[r] * v)
        if not store_early:
            keep()
    if g == 0:
        out["e"][n - 2] = x[n - 1]
    if n - 1 in A:
        out["d"][n - 1] = A[n - 1][n - 1]


def reduce_with_late(M, G, late, store_early=False):
    S, n, slots = M.copy(), len(M), {}
    out = dict(d=np.zeros(n), e=np.zeros(n - 1), beta=np.zeros(n))
    out["d"][0] = M[0, 0]
    waiting = [workgroup(g, G, S, slots, out, store_early) for g in range(G) if g != late]
    if late is not None:
        for w in waiting:  # (to their first wait)
            next(w)
        waiting.insert(0, workgroup(late, G, S, slots, out, store_early))
    while waiting:
        waiting = [w for w in waiting if next(w, "end") != "end"]
    return np.concatenate([out["d"], out["e"], out["beta"], np.triu(S, 1).ravel()]), out


@pytest.mark.parametrize("n,rows", [(33, 8), (50, 16), (41, 32)])
def test_results_do_not_depend_on_when_a_workgroup_starts(n, rows):
    M = np.random.default_rng(n).standard_normal((n, n))
    M = M + M.T
    G = -(-n // rows)
    ref, out = reduce_with_late(M, G, None)
    T = np.diag(out["d"]) + np.diag(out["e"], 1) + np.diag(out["e"], -1)
    # backward error of a Householder reduction: a few n roundings of the norm
    assert np.max(np.abs(np.linalg.eigvalsh(T) - np.linalg.eigvalsh(M))) <= 10 * n * 2.2e-16 * np.abs(M).sum(0).max()
    for late in range(G):
        assert np.array_equal(reduce_with_late(M, G, late)[0], ref), late
    for late in range(1, G):  # (workgroup 0 stores row 0 itself)
        assert not np.array_equal(reduce_with_late(M, G, late, store_early=True)[0], ref), late
