"""GPU: a gcd works in the workspace that its column sums need (the sizes below), with
the same results as in a large one, and is refused in half of it."""

import pytest

from oracle.poly import pmul
from workloads import rng_for

pytestmark = pytest.mark.gpu


def dense(part, deg, bits):
    rng = rng_for(992, part)
    v = [int(x) for x in rng.integers(-(1 << bits), 1 << bits, size=deg + 1)]
    v[deg] = v[deg] or 1
    v[0] = v[0] or 1
    return v


def operands(da, db, dg, bits):
    g = dense(500 + da, dg, bits)
    return pmul(dense(501 + da, da, bits), g), pmul(dense(502 + da, db, bits), g)


def wide_operands():
    u, v = ([x << 15000 for x in dense(p, d, 60)] for p, d in ((700, 12), (701, 10)))
    u[0] += 1
    v[0] += 1
    return u, v


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


@pytest.fixture(scope="module")
def big(rsl):
    c = rsl.Context(device=0, workspace_bytes=1 << 28)
    yield c
    c.close()


@pytest.mark.parametrize("shape,need", [((3, 2, 2, 20), 9280), ((60, 50, 0, 20), 29184), ((60, 50, 10, 40), 43840),
                                        ((250, 200, 100, 20), 354432), ((200, 200, 150, 62), 482944),
                                        ((5, 200, 10, 20), 62720), ("wide", 5918912)])
def test_least_workspace(rsl, big, shape, need):
    u, v = wide_operands() if shape == "wide" else operands(*shape)
    want = big.gcd(u, v)
    g, a, b = want
    assert pmul(g, a) == u and pmul(g, b) == v
    ctx = rsl.Context(device=0, workspace_bytes=need, table_bytes=128 << 20)
    assert ctx.gcd(u, v) == want
    assert ctx.last_error() == ""
    ctx.close()
    ctx = rsl.Context(device=0, workspace_bytes=need // 2, table_bytes=128 << 20)
    with pytest.raises(rsl.RSLError) as e:
        ctx.gcd(u, v)
    assert e.value.code == rsl.RSL_ENOMEM
    ctx.close()
