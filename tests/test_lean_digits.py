"""Problems of low degree over hundreds of primes, whose CRT digits take more memory
than their layouts spare elsewhere.  CPU: a call needs no more than the column
layout with column sums (the sizes below).  GPU: calls, jobs, a batch and a server
in that memory give the bits of the usual layout."""

import pytest

from workloads import rng_for, small_random

SHAPES = [((17, 1), (49, 2), 219, 4311808), ((22, 2), (9, 2), 425, 2426112), ((44, 1), (52, 1), 131, 4839168),
          ((6, 1), (53, 3), 194, 2973952), ((3, 2), (2, 3), 1500, 1746176), ((9, 9), (9, 9), 512, 8404992)]


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


def operands(shape):
    (a, b), (c, d), bits, _ = shape
    rng = rng_for(987, a)
    return small_random(rng, a, b, bits), small_random(rng, c, d, bits)


@pytest.mark.parametrize("shape", SHAPES)
def test_query_footprint(rsl, shape):
    assert rsl.query(*operands(shape))["footprint_bytes"] <= shape[-1]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES[:4])
def test_least_memory(rsl, shape):
    f, g = operands(shape)
    big = rsl.Context(device=0, workspace_bytes=1 << 28)
    want = big.res(f, g)
    usual = big.job([(f, g, "y")])
    need = rsl.query(f, g)["footprint_bytes"]
    assert need < usual.info()["device_bytes"]
    usual.close()
    ctx = rsl.Context(device=0, workspace_bytes=need)
    assert ctx.res(f, g) == want
    assert ctx.res(f, g, prime_start=0) == want
    assert ctx.batch([(f, g, "y")], mode="plain") == [want]
    job = big.job([(f, g, "y")], device_bytes=need)
    for mode, graph in (("staged", False), ("plain", False), ("staged", True), ("staged", True)):
        job.run(mode, graph=graph)
        assert job.results() == [want], mode
    job.close()
    # a prime list of its own (Garner's tables in the image, as an undecided quotient needs)
    own = big.job([(f, g, "y")], prime_start=3, device_bytes=shape[-1] + (4 << 20))
    own.run("staged")
    assert own.results() == [want]
    own.close()
    ctx.close()
    big.close()


@pytest.mark.gpu
def test_batch_and_server(rsl):
    probs = [(*operands(s), "y") for s in SHAPES[:4]]
    big = rsl.Context(device=0, workspace_bytes=1 << 28)
    want = big.batch(probs, mode="staged")
    total = sum(s[-1] for s in SHAPES[:4])
    ctx = rsl.Context(device=0, workspace_bytes=total)
    assert ctx.batch(probs, mode="staged") == want
    assert ctx.batch(probs, mode="plain") == want
    srv = rsl.Server(ctx, budget_bytes=total, max_slots=8)
    tickets = [srv.submit(*p) for p in probs + probs]
    assert [srv.wait(t, timeout_ms=60000) for t in tickets] == want + want
    srv.close()
    ctx.close()
    big.close()
