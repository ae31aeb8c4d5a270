"""The dense calls when the one-launch tridiagonal reduction gives up (its workgroups are not all on the
chip, e.g. beside another process's): the library solves again with the reduction by launches a step.
Forced by a context whose reductions may not poll at all, so that every workgroup leaves at its first
wait; and the reduction by launches alone (no one-launch reduction before it) gives the same bits.

Against the one-launch results: roots 1e-9, energies 1e-10 Ha (1e-9 above n = 513), NTO weights 1e-12 of
the largest, as the tests of these calls against the oracle; vectors up to the same bound times the
inverse of the least root distance, 1e-7."""
import ctypes

import numpy as np
import pytest

from workloads import gen
import paper_2512_12515_amd as P

pytestmark = pytest.mark.gpu


def set_polls(ctx, polls):
    fn = P.binding.lib().pprpa_test_tridiagonal_polls
    fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_int32], ctypes.c_int
    assert fn(ctx._h, polls) == P.binding.OK


def in_each_form(ctx, call):
    """The call's arrays in one launch, after it gave up, and by launches alone."""
    out = [call()]
    for polls in (0, -1):
        set_polls(ctx, polls)
        out.append(call())
    return out


@pytest.mark.parametrize("nocc,nvir,n", [(3, 13, 97), (5, 20, 225), (2, 31, 499), (12, 32, 606),
                                         (32, 33, 1089)])
def test_dense_solves(nocc, nvir, n):
    eps, L = gen.orbital_energies(81, nocc, nvir), gen.lpq_full(81, nocc + nvir, 60)
    with P.PpRPA(eps, L, nocc, mult="singlet", dense=True) as ctx:
        assert ctx.n == n

        def solve():
            print("dense fallback", n, flush=True)
            out = []
            for channel in ("pp", "hh"):
                r = ctx.davidson(min(3, ctx.n_hh), direct=True, vectors=True, channel=channel)
                out += [r["omega"], r["vecs"]]
            for noalloc in (False, True)[:1 + (n <= 512)]:
                out.append(np.array(list(ctx.correlation_energy(noalloc=noalloc).values())))
            return out

        one, gave_up, launches = in_each_form(ctx, solve)
    for i, (a, b, c) in enumerate(zip(one, gave_up, launches)):
        assert np.array_equal(b, c), i
        tol = 1e-7 if i in (1, 3) else 1e-9 if i < 4 or n > 513 else 1e-10
        assert np.max(np.abs(a - b)) <= tol, i


@pytest.mark.parametrize("nocc,nvir,k", [(3, 4, 3), (3, 33, 5), (20, 200, 3), (1, 257, 3)])
def test_nto_weights(nocc, nvir, k):
    eps, L = gen.orbital_energies(82, nocc, nvir), gen.lpq_full(82, nocc + nvir, 8)
    with P.PpRPA(eps, L, nocc, mult="singlet") as ctx:
        z = gen.random_vectors(83, k, ctx.n)
        check_nto(ctx, z)


def test_nto_weights_alpha_beta():
    nmo, noa, nob = 60, 9, 7
    ea, eb = gen.orbital_energies(84, noa, nmo - noa), gen.orbital_energies(85, nob, nmo - nob)
    with P.PpRPA.alpha_beta(ea, eb, gen.lpq_full(84, nmo, 8), gen.lpq_full(85, nmo, 8), noa, nob,
                            density_fitted=True) as ctx:
        check_nto(ctx, gen.random_vectors(86, 4, ctx.n))


def check_nto(ctx, z):
    def call():
        print("nto fallback", ctx.nv, ctx.no, flush=True)
        r = ctx.nto(z)
        return [r[key] for key in sorted(r)]

    one, gave_up, launches = in_each_form(ctx, call)
    for a, b, c in zip(one, gave_up, launches):
        assert np.array_equal(b, c)
        assert np.max(np.abs(a - b)) <= 1e-12 * max(np.abs(a).max(), 1e-300)


def test_stream_with_a_part_of_the_compute_units():
    """A context on a stream that may use half of the compute units reduces by launches a step, at once."""
    import time

    import torch
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so.7")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    mask = (ctypes.c_uint32 * ((cus + 31) // 32))(*[0xFFFFFFFF] * (cus // 64))  # the first half
    stream = ctypes.c_void_p()
    hip.hipExtStreamCreateWithCUMask.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint32,
                                                 ctypes.POINTER(ctypes.c_uint32)]
    hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    rc = hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), len(mask), mask)
    if rc != 0:
        torch.cuda.synchronize()
        pytest.skip(f"no stream with a compute unit mask here (HIP error {rc})")
    nocc, nvir = 12, 32
    eps, L = gen.orbital_energies(87, nocc, nvir), gen.lpq_full(87, nocc + nvir, 60)

    def solve(ctx):
        r = ctx.davidson(3, direct=True, vectors=True)
        return [r["omega"], r["vecs"], np.array(list(ctx.correlation_energy().values()))]

    try:
        with P.PpRPA(eps, L, nocc, dense=True) as ctx:
            set_polls(ctx, -1)
            ref = solve(ctx)
        with P.PpRPA(eps, L, nocc, dense=True, stream=stream.value) as ctx:
            solve(ctx)
            print("dense on a part of the compute units", flush=True)
            t = time.perf_counter()
            got = solve(ctx)
            t = time.perf_counter() - t
    finally:
        assert hip.hipStreamDestroy(stream) == 0
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    assert t < 1.0  # (a reduction that waits in vain takes seconds)
