"""GPU: long coefficients through the two-limb reduction steps, at every parity
of the limb count around its chunks of 16, with limbs at the ends of their
signed and unsigned ranges, against the oracle."""

import random

import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1010_1386_amd as rsl
    c = rsl.Context(device=0, workspace_bytes=1 << 28)
    yield c
    c.close()


def extremes(L):
    """Values of exactly L limbs (two's complement) with limbs of one pattern."""
    top = 1 << (32 * L - 1)
    out = [top - 1, -top, -top + 1, 1 - top]
    for w in (0x7FFFFFFF, 0x80000000, 0xFFFFFFFF, 0x00000001):
        v = sum(w << (32 * i) for i in range(L - 1))
        out += [v + (1 << (32 * L - 2)), -v - (1 << (32 * L - 2))]
    return out


@pytest.mark.parametrize("L", [3, 4, 5, 15, 16, 17, 18, 19, 32, 33, 34, 48, 49, 50])
def test_limb_counts(ctx, L):
    rnd = random.Random(L)
    ex = extremes(L)
    pick = lambda: rnd.choice(ex + [0, 1, -1, rnd.getrandbits(32 * L - 1)])
    for d in (1, 9):  # one K run per row; two, the second with one coefficient
        F = [[pick() for _ in range(d)], [pick() for _ in range(d - 1)] + [ex[L % len(ex)]]]
        G = [[pick() for _ in range(d)], [ex[0]]]
        assert ctx.res(F, G) == oracle.res(F, G)
