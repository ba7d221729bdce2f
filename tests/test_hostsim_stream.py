"""CPU check of the streamed register form (csrc/ures_regs.h, ures_stream: signed
residues, the longer polynomial divided from memory by the shorter one in
registers) against the oracle's determinant mod p: every residue of the shorter
degree modulo 4, equal and very unequal degrees, both orders, extreme residues,
vanishing leading coefficients, common factors and degree drops."""

import ctypes

import pytest

from oracle import det_mod
from test_hostsim_ures import LIB, PRIMES, hs  # noqa: F401  (builds the library when a source is newer)
from workloads import rng_for


def stream(nmax, p, A, B):
    lib = ctypes.CDLL(LIB)
    a, b = (ctypes.c_uint32 * len(A))(*A), (ctypes.c_uint32 * len(B))(*B)
    out, bad, gen = ctypes.c_uint32(), ctypes.c_int(), ctypes.c_int()
    rc = lib.hs_ures_stream(nmax, ctypes.c_uint32(p), len(A) - 1, len(B) - 1, a, b, ctypes.byref(out),
                            ctypes.byref(bad), ctypes.byref(gen))
    assert rc == 0
    return out.value, bool(bad.value), bool(gen.value)


def sylvester(A, B, p):
    """The determinant of the Sylvester matrix with the formal degrees, mod p."""
    m, n = len(A) - 1, len(B) - 1
    rows = [[0] * i + A[::-1] + [0] * (n - 1 - i) for i in range(n)]
    rows += [[0] * i + B[::-1] + [0] * (m - 1 - i) for i in range(m)]
    return det_mod(rows, p)


SHAPES = [(8, 1, 1), (8, 5, 1), (8, 2, 2), (8, 3, 4), (8, 8, 8), (8, 7, 30), (16, 9, 9), (16, 12, 10), (16, 16, 15),
          (16, 11, 40), (24, 17, 17), (24, 24, 23), (24, 43, 19), (32, 32, 32), (32, 25, 31), (40, 33, 34),
          (40, 42, 40), (48, 41, 42), (48, 48, 48), (48, 45, 63), (48, 7, 6)]


@pytest.mark.parametrize("nmax,m,n", SHAPES)
def test_stream_matches_determinant(hs, nmax, m, n):  # noqa: F811
    rng = rng_for(910, nmax, 100 * m + n)
    for p in PRIMES:
        for A, B in [([int(v) for v in rng.integers(0, p, m + 1)], [int(v) for v in rng.integers(0, p, n + 1)]),
                     ([p - 1] * (m + 1), [p // 2 + (j & 1) for j in range(n + 1)]),
                     ([(p + 1) // 2 - (j & 1) for j in range(m + 1)], [int(v) for v in rng.integers(0, p, n + 1)])]:
            got, bad, _ = stream(nmax, p, A, B)
            assert got == sylvester(A, B, p) and not bad
        # random coefficients: the generic pattern itself (a drop has probability ~ n / p)
        A, B = ([int(v) for v in rng.integers(1, p, d + 1)] for d in (m, n))
        assert stream(nmax, p, A, B)[2]


def test_stream_leaves_the_generic_pattern(hs):  # noqa: F811
    p = PRIMES[0]
    rng = rng_for(911, 0)
    mul = lambda f, g: [sum(f[i] * g[k - i] for i in range(len(f)) if 0 <= k - i < len(g)) % p  # noqa: E731
                        for k in range(len(f) + len(g) - 1)]
    r = lambda d: [int(v) for v in rng.integers(1, p, d + 1)]  # noqa: E731
    for A, B, bad, generic in [
            (r(9) + [0], r(9), True, False), (r(9), r(9) + [0], True, False), (r(4) + [0], r(6) + [0], True, False),
            (mul(r(2), r(6)), mul(r(0), r(7)), False, True),
            ([5, 0, 0, 7, 0, 0, 1], [3, 0, 0, 1], False, False), ([1, 0, 3, 0, 9], [2, 0, 1], False, False)]:
        got, b, g = stream(16, p, A, B)
        assert got == sylvester(A, B, p) and b == bad and g == generic
    h = r(3)  # a common factor of degree 3, and of degree 1 (the constant remainder vanishes)
    assert stream(16, p, mul(h, r(5)), mul(h, r(4)))[0] == 0
    h = r(1)
    assert stream(16, p, mul(h, r(7)), mul(h, r(7)))[0] == 0
