"""GPU: the CRT on the matrix cores against closed forms and Garner's digits
(RSL_CRT_GARNER, the column-sum kernel): prime counts around its 64-prime slices
and around every row-tile choice, coefficient counts around its items, and
coefficients next to +-(M - 1) / 2, whose quotient the fixed-point estimate cannot
decide."""

import math
import os

import pytest

from workloads import _uniform_signed, dense_total, rng_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1010_1386_amd as m
    c = m.Context(device=0, workspace_bytes=1 << 30)
    yield c
    c.close()


@pytest.fixture(scope="module")
def garner():
    import paper_1010_1386_amd as m
    os.environ["RSL_CRT_GARNER"] = "1"
    try:
        c = m.Context(device=0, workspace_bytes=1 << 30)
    finally:
        del os.environ["RSL_CRT_GARNER"]
    yield c
    c.close()


def primes(n):
    """The first n primes below 2^32 / 3, descending (Miller-Rabin, exact below 2^32)."""
    def is_prime(q):
        d, s = q - 1, 0
        while d % 2 == 0:
            d, s = d // 2, s + 1
        for a in (2, 3, 5, 7):
            x = pow(a, d, q)
            if x in (1, q - 1):
                continue
            for _ in range(s - 1):
                x = x * x % q
                if x == q - 1:
                    break
            else:
                return False
        return True
    out, q = [], (1 << 32) // 3 | 1
    while len(out) < n:
        if is_prime(q):
            out.append(q)
        q -= 2
    return out


@pytest.mark.parametrize("np_", [1, 2, 3, 40, 63, 64, 65, 128, 129, 257, 512])
def test_undecided_quotients(ctx, garner, np_):
    """res_y(a y + b, -b y + a) = a^2 + b^2 just below M / 2 (and its negative):
    the Hadamard bound is attained, so the planner takes exactly np_ primes."""
    import paper_1010_1386_amd as rsl
    M = math.prod(primes(np_))
    H = (M - 1) // 2
    a = math.isqrt(H)
    b = math.isqrt(H - a * a)
    assert 0 <= (H - a * a - b * b) << 34 < M or np_ == 1
    for f, g, want in [([[b], [a]], [[a], [-b]], a * a + b * b), ([[a], [-b]], [[b], [a]], -(a * a + b * b))]:
        assert rsl.query(f, g)["n_primes"] == np_
        assert ctx.res(f, g) == [want]
        assert garner.res(f, g) == [want]


@pytest.mark.parametrize("extra", [0, 61, 62, 63, 125, 126, 253, 254, 509])
def test_prime_counts(ctx, garner, extra):
    rng = rng_for(970, extra)
    p, q = _uniform_signed(rng, 40, 40), _uniform_signed(rng, 40, 33)
    f, g = [p, [7] + [0] * 39], [q, [-3] + [0] * 32]
    want = [7 * (q[i] if i < 33 else 0) + 3 * p[i] for i in range(40)]
    assert ctx.res(f, g, extra_primes=extra) == want
    assert garner.res(f, g, extra_primes=extra) == want


@pytest.mark.parametrize("count,shift", [(60, 0), (100, 0), (200, 0), (100, 1300), (200, 3000)])
def test_row_tiles(ctx, garner, count, shift):
    """Jobs of few and of many coefficients, few and many primes (all row-tile choices)."""
    rng = rng_for(971, count, shift)
    probs, want = [], []
    for k in range(count):
        D = [255, 256, 257, 15, 16, 17, 700][k % 7]
        p, q = _uniform_signed(rng, 30, D + 1), _uniform_signed(rng, 30, D + 1)
        s = shift if k == 3 else 0
        probs.append(([[v << s for v in p], [5] + [0] * D], [q, [2] + [0] * D], "y"))
        R = [5 * q[i] - 2 * (p[i] << s) for i in range(D + 1)]
        while R and R[-1] == 0:
            R.pop()
        want.append(R)
    for c in (ctx, garner):
        job = c.job(probs)
        for mode in ("staged", "plain"):
            job.run(mode)
            assert job.results() == want, mode
        job.close()


def test_wide_beside_slots(ctx, garner):
    """A problem of more than 512 primes in one job with small ones."""
    rng = rng_for(972, 0)
    big = [[int(v) << 900 for v in row] for row in dense_total(rng, 9, 20)]
    probs = [(big, dense_total(rng, 9, 20), "y"), (dense_total(rng, 5, 20), dense_total(rng, 4, 20), "y")]
    out = []
    for c in (ctx, garner):
        job = c.job(probs, extra_primes=300)
        job.run("staged")
        out.append(job.results())
        job.close()
    assert out[0] == out[1]
