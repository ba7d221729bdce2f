"""GPU: calls whose usual layout does not fit the memory they have are laid out with
the least memory (digit tiles only within the column layout's footprint) and give
the same bits: a workspace of exactly the queried footprint, a job bound to
exactly that, a server budget of exactly that, for shapes whose digit tiles are
larger than their column layouts."""

import pytest

from workloads import rng_for, small_random

pytestmark = pytest.mark.gpu

SHAPES = [(2, 33, 3, 9), (45, 5, 11, 1), (33, 6, 6, 33), (47, 45, 3, 3), (8, 8, 8, 8)]


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


@pytest.fixture(scope="module")
def big(rsl):
    c = rsl.Context(device=0, workspace_bytes=1 << 30)
    yield c
    c.close()


@pytest.mark.parametrize("shape", SHAPES)
def test_exact_footprint(rsl, big, shape):
    rng = rng_for(980, *shape[:2])
    a, b, c, d = shape
    f, g = small_random(rng, a, b, 30), small_random(rng, c, d, 30)
    need = rsl.query(f, g)["footprint_bytes"]
    want = big.res(f, g)
    ctx = rsl.Context(device=0, workspace_bytes=need)
    assert ctx.res(f, g) == want
    assert ctx.batch([(f, g, "y")], mode="batched") == [want]
    assert ctx.batch([(f, g, "y")], mode="staged") == [want]
    srv = rsl.Server(ctx, budget_bytes=need, max_slots=4)
    try:
        t = [srv.submit(f, g, "y") for _ in range(2)]
        assert [srv.wait(x, timeout_ms=60000) for x in t] == [want] * 2
    except rsl.RSLError as e:  # the server's layout may need more than a call's
        assert e.code == rsl.RSL_ENOMEM
    srv.close()
    ctx.close()
    job = big.job([(f, g, "y")], device_bytes=need)
    for mode in ("staged", "batched", "plain", "staged"):
        job.run(mode)
        assert job.results() == [want], mode
    job.close()


def test_schedules_share_memory(big):
    """Digit tiles and the persistent schedule's buffers share memory: runs of the
    schedules in turn, with graph replays between them."""
    rng = rng_for(981, 0)
    probs = [(small_random(rng, 9 + k, 7 + 3 * k, 20), small_random(rng, 8, 35 - 2 * k, 20), "yx"[k % 2])
             for k in range(8)]
    job = big.job(probs)
    job.run("staged")
    want = job.results()
    for mode, graph in [("batched", False), ("staged", False), ("staged", True), ("batched", True), ("staged", True),
                        ("plain", False), ("batched", False), ("plain", True), ("staged", True)]:
        job.run(mode, graph=graph)
        assert job.results() == want, (mode, graph)
    job.close()
