"""GPU parity with the oracle on finite matrices whose elimination overflows:
infinities and NaN appear in the columns still to be searched, and pivots,
info, factors and solution follow the oracle's scan (a candidate replaces the
best so far only if its magnitude is larger, so NaN never does)."""
import numpy as np
import pytest

import oracle
from test_gpu_lupp import gpu_solve, variants

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2609_15217_amd.lupp as L
    return L


@pytest.fixture(scope="module")
def ctx(L):
    return L.Context(0)


def overflowing(n, count, seed):
    """Entries up to 1.9 * 2^1023; every third system with zeros, every third
    with rows of 2^-40 times that."""
    r = np.random.default_rng(seed)
    A = np.ldexp(np.clip(r.standard_normal((count, n, n)), -1.9, 1.9), 1023)
    A[1::3][r.random(A[1::3].shape) < 0.4] = 0.0
    A[2::3] *= np.where(r.random((len(A[2::3]), n, 1)) < 0.5, 1.0, 2.0 ** -40)
    b = np.ldexp(r.uniform(-1, 1, (count, n)), 1000)
    assert np.isfinite(A).all()
    return A, b


def check(ref, LU, x, pv, io, b):
    assert np.array_equal(io, ref["info"])
    assert np.array_equal(pv, ref["ipiv"])
    assert np.array_equal(LU, ref["LU"], equal_nan=True)
    ok = ref["info"] == 0
    assert np.array_equal(x[ok], ref["x"][ok], equal_nan=True)
    assert np.array_equal(x[~ok], b[~ok])


@pytest.mark.parametrize("n", list(range(2, 14)))
def test_thread_solver(L, ctx, n):
    A, b = overflowing(n, 300, seed=9000 + n)
    for fma in (False, True):
        ref = oracle.gesv_batch_mode(A, b, fma=fma, threads=4)
        for layout in (L.LUPP_AOS, L.LUPP_SOA):
            got = gpu_solve(L, ctx, A, b, layout, L.LUPP_VARIANT_THREAD, 1, fma=fma)
            check(ref, *got[:4], b)


@pytest.mark.parametrize("n", [2, 4, 5, 8, 9, 12, 13, 16, 17, 20, 24, 25, 32])
def test_lanes_solver(L, ctx, n):
    A, b = overflowing(n, 300, seed=9100 + n)
    for fma in (False, True):
        ref = oracle.gesv_batch_mode(A, b, fma=fma, threads=4)
        for variant, lanes in variants(n):
            if variant != L.LUPP_VARIANT_LANES:
                continue
            for layout in (L.LUPP_AOS, L.LUPP_SOA):
                got = gpu_solve(L, ctx, A, b, layout, variant, lanes, fma=fma)
                check(ref, *got[:4], b)
