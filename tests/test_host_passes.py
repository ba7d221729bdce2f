"""The host's passes over a call's limbs.  CPU: primes that divide the leading
coefficient at the edges of the blocks they are tested in, and rows at the edge
of the 128-bit norm sums, against exact integers.  GPU: results taken in blocks
of coefficients into rows of the bound's width, wider ones, exactly the needed
one, and one too narrow (refused, nothing written)."""

import contextlib
import ctypes
import math

import numpy as np
import pytest

import oracle
from workloads import dense_total, rng_for


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


def _table_primes(n):
    # the library's table: the primes below 2^32 / 3, descending
    return oracle.next_check_primes(n, below=(1 << 32) // 3 + 1)


@pytest.mark.parametrize("bad", [[0], [7], [8], [6, 7, 8, 9], [0, 15, 16], [3, 11]])
def test_bad_primes_at_block_edges(rsl, bad):
    ps = _table_primes(20)
    q = math.prod(ps[k] for k in bad)
    big = 1 << 300
    F = [[1, 2, big + 5], [5, 0, 1], [3 * q, -2 * q]]
    G = [[2, 1], [1, 1, 1], [big + 3]]
    for f, g in ((F, G), (G, F)):
        r = rsl.query(f, g, "y")
        assert r["bad_primes"] == len(bad)
        used = r["n_primes"]
        M = math.prod(p for p in _table_primes(used + len(bad)) if q % p)
        B2 = oracle.hadamard_bound_sq(f, g, "y")
        assert M * M > 4 * B2 and r["out_limbs"] == (M.bit_length() + 31) // 32
    # one coefficient of the leading row is coprime to the primes: none is bad
    F[2][1] = 7
    assert rsl.query(F, G, "y")["bad_primes"] == 0


@pytest.mark.parametrize("row", [(1 << 60) - 1, 1 << 60, (1 << 63) - 1, -(1 << 63), (1 << 31) - 1])
def test_norms_at_128_bits(rsl, row):
    F = [[row, row], [1, row], [row, row, row], [3]]
    G = [[row], [2], [row, -1], [1, 1]]
    for var in "yx":
        r = rsl.query(F, G, var)
        B2 = oracle.hadamard_bound_sq(F, G, var)
        ps = _table_primes(r["n_primes"] + r["bad_primes"])
        M = math.prod(ps)
        assert r["bad_primes"] == 0
        assert M * M > 4 * B2 and (M // ps[-1]) ** 2 <= 4 * B2


@pytest.mark.gpu
def test_result_rows_of_every_width(rsl):
    rng = rng_for(930, 1)
    with contextlib.closing(rsl.Context(device=0, workspace_bytes=1 << 28)) as ctx:
        for d, bits in ((3, 6), (26, 40)):  # a block; several of about 64 KiB
            F, G = dense_total(rng, d, bits), dense_total(rng, d, bits)
            q = rsl.query(F, G, "y")
            D, L = q["D"], q["out_limbs"]
            if d == 26:
                assert (D + 1) * L > 2 * (1 << 14)
            want = ctx.res(F, G)
            pf, pg = rsl.Poly(F), rsl.Poly(G)
            # sign-extended limbs of the widest coefficient
            need = max((c if c >= 0 else ~c).bit_length() // 32 + 1 for c in want)
            for limbs in (L + 3, L, need, need - 1):
                buf = np.full((D + 1) * max(limbs, 1), 0xA5A5A5A5, dtype=np.uint32)
                out = rsl.rsl_result(D, limbs, buf.ctypes.data_as(ctypes.POINTER(ctypes.c_uint32)), 0, 0)
                rc = rsl._lib.rsl_res(ctx.h, ctypes.byref(pf.c), ctypes.byref(pg.c), 0, None, ctypes.byref(out))
                assert (out.deg, out.needed_limbs) == (len(want) - 1, need)
                if limbs < need:
                    assert rc == rsl.RSL_ERANGE and (buf == 0xA5A5A5A5).all()
                    continue
                assert rc == 0
                rows = buf.reshape(D + 1, limbs)
                got = [int.from_bytes(rows[k].tobytes(), "little", signed=True) for k in range(len(want))]
                assert got == want
