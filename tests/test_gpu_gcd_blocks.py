"""GPU: the modular gcd's blocks at the edges of their 64-lane waves and 256
threads: degree pairs around both, remainder sequences with gaps (several
eliminations in one division, a remainder that drops by more than one degree),
and a constant or equal second operand, against the oracle."""

import random

import pytest

from oracle.poly import pmul, ptrim
from oracle.sqfree import zx_divexact, zx_gcd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1010_1386_amd as rsl
    c = rsl.Context(device=0, workspace_bytes=1 << 28)
    yield c
    c.close()


def dense(rnd, deg):
    return [rnd.randint(-3, 3) for _ in range(deg)] + [rnd.choice([1, -1, 2])]


def sparse(deg, *low):
    c = [0] * (deg + 1)
    c[deg] = 1
    for k, v in low:
        c[k] = v
    return c


@pytest.mark.parametrize("du,dv", [(1, 1), (2, 1), (63, 62), (64, 64), (65, 63), (128, 3), (255, 254), (256, 1),
                                   (257, 256), (258, 130)])
@pytest.mark.parametrize("dc", [0, 1, 5])
def test_degrees_at_the_edges(ctx, du, dv, dc):
    """u = c a and v = c b: a and b chosen so that the oracle's gcd is cheap (b
    sparse), the common factor c known."""
    rnd = random.Random(1000 * du + 10 * dv + dc)
    c = dense(rnd, dc) if dc else [1]
    a = sparse(du, (0, -1), (min(1, du - 1), 3)) if du > 1 else [3, 1]
    b = sparse(dv, (0, 2)) if dv > 1 else [1, 2]
    u, v = ptrim(pmul(a, c)), ptrim(pmul(b, c))
    g, p, q = ctx.gcd(u, v)
    assert pmul(g, p) == u and pmul(g, q) == v
    if du <= 65:
        assert g == zx_gcd(u, v)
    elif dc:
        cc = c if c[-1] > 0 else [-x for x in c]
        zx_divexact(g, cc)  # raises or leaves a remainder unless c divides g


@pytest.mark.parametrize("u,v", [
    (sparse(64, (0, -1)), sparse(48, (0, -1))),    # x^16 - 1: every division has a gap
    (sparse(257, (0, 1)), sparse(255, (3, 1))),    # remainders that drop by many degrees
    (sparse(130, (65, 2), (0, 1)), [7]),
    (sparse(256, (0, 5)), sparse(256, (0, 5))),
])
def test_gaps(ctx, u, v):
    g, p, q = ctx.gcd(u, v)
    assert pmul(g, p) == u and pmul(g, q) == v
    assert g == zx_gcd(u, v)
