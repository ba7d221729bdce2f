"""GPU: the limb digits of M / p_i formed from M alone, at the edges of their
blocks of 64 primes and 64 limbs and from prime lists that start anywhere: a
small resultant over far more primes than it needs equals the one over its own
primes (and the vector-ALU sums, which read the M_i of the host)."""

import pytest

from workloads import dense_total, rng_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


@pytest.mark.parametrize("start", [0, 5])
@pytest.mark.parametrize("np", [513, 528, 576, 577, 640, 661, 662, 1057])
def test_block_edges(rsl, monkeypatch, np, start):
    rng = rng_for(931, np)
    F, G = dense_total(rng, 3, 20), dense_total(rng, 2, 20)
    extra = np - rsl.query(F, G, "y")["n_primes"]
    ctx = rsl.Context(device=0, workspace_bytes=1 << 28)
    want = ctx.res(F, G)
    assert ctx.res(F, G, extra_primes=extra, prime_start=start) == want
    ctx.close()
    monkeypatch.setenv("RSL_WIDE_VALU", "1")
    ctx = rsl.Context(device=0, workspace_bytes=1 << 28)
    assert ctx.res(F, G, extra_primes=extra, prime_start=start) == want
    ctx.close()
