"""GPU: the staged and plain runs against paths that share neither their interpolation
nor their layout: the persistent schedule (vector-ALU convolution and basis change),
divided differences for every prime (interp_newton), and the oracle -- single
problems, both projections, bad points and formal points, multi-limb inputs, a shifted
origin, a batch sharing primes.  And a server whose budget is exactly what it plans for
a request, for shapes whose usual layouts need more."""

import ctypes

import pytest

import oracle
from test_gpu_lean_layout import SHAPES
from workloads import dense_total, rng_for, small_random

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(rsl):
    c = rsl.Context(device=0, workspace_bytes=1 << 30)
    yield c
    c.close()


def everyway(ctx, probs, **opts):
    """The results of a job in every schedule, with divided differences, and with whole sums."""
    out = []
    for o, modes in ((opts, ("staged", "plain", "batched")), (dict(opts, interp_newton=True), ("staged", "batched")),
                     (dict(opts, interp_mm=True), ("batched", "staged"))):
        job = ctx.job(probs, **o)
        for mode in modes:
            job.run(mode)
            out.append(((mode, o), job.results()))
        job.close()
    for way, got in out[1:]:
        assert got == out[0][1], way
    return out[0][1]


def test_single_problems_and_pairs(ctx):
    rng = rng_for(988, 0)
    for k in range(8):
        F = dense_total(rng, int(rng.integers(2, 9)), int(rng.integers(8, 64)))
        G = dense_total(rng, int(rng.integers(2, 9)), int(rng.integers(8, 64)))
        want = [oracle.res(F, G, v) for v in "yx"]
        assert everyway(ctx, [(F, G, "y")]) == want[:1]
        assert everyway(ctx, [(F, G, "y"), (F, G, "x")]) == want


def test_bad_points_origins_and_limbs(ctx):
    rng = rng_for(988, 1)
    F = small_random(rng, 4, 5, 40)
    F[4] = [0, -2, 1, 0, 0, 0]  # lc_y = x (x - 2): points 0 and 2 are bad for every prime
    G = small_random(rng, 3, 4, 40)
    want = [oracle.res(F, G, "y")]
    for opts in ({}, {"points": "formal"}, {"point_origin": -1}, {"point_origin": 9}, {"extra_points": 7},
                 {"prime_start": 2}):
        assert everyway(ctx, [(F, G, "y")], **opts) == want, opts
    big = [[int(v) << 180 for v in row] for row in small_random(rng, 5, 5, 30)]
    G2 = small_random(rng, 4, 4, 30)
    assert everyway(ctx, [(big, G2, "y"), (big, G2, "x")]) == [oracle.res(big, G2, v) for v in "yx"]


def test_batch_sharing_primes(ctx):
    rng = rng_for(988, 2)
    probs = []
    for k in range(24):
        F = dense_total(rng, int(rng.integers(2, 14)), int(rng.integers(8, 48)))
        G = dense_total(rng, int(rng.integers(2, 14)), int(rng.integers(8, 48)))
        if k % 7 == 3:
            F[-1] = [0, -3, 1]  # a non-constant leading coefficient: bad points
        probs.append((F, G, "yx"[k % 2]))
    got = everyway(ctx, probs)
    for k in range(0, 24, 5):
        assert got[k] == oracle.res(*probs[k]), k


@pytest.mark.parametrize("shape", SHAPES)
def test_server_in_its_own_footprint(rsl, ctx, shape):
    rng = rng_for(988, 3 + shape[0])
    a, b, c, d = shape
    f, g = rsl.Poly(small_random(rng, a, b, 30)), rsl.Poly(small_random(rng, c, d, 30))
    want = ctx.res(f, g)
    own = rsl.Context(device=0, workspace_bytes=64 << 20)

    def planned(srv):
        info, handle = rsl.rsl_info(), ctypes.c_uint64()
        assert rsl._lib.rsl_server_plan(srv.h, ctypes.byref(f.c), ctypes.byref(g.c), rsl.RSL_Y, ctypes.byref(info),
                                        ctypes.byref(handle)) == 0
        return info.footprint_bytes

    srv = rsl.Server(own, budget_bytes=64 << 20)
    need = planned(srv)
    srv.close()
    srv = rsl.Server(own, budget_bytes=need, max_slots=4)
    assert planned(srv) == need
    tickets = [srv.submit(f, g, "y") for _ in range(3)]
    assert [srv.wait(t, timeout_ms=60000) for t in tickets] == [want] * 3
    assert srv.stats()["max_batch"] == 1 and srv.stats()["admitted_bytes_peak"] <= need
    srv.close()
    srv = rsl.Server(own, budget_bytes=need - 1)
    with pytest.raises(rsl.RSLError) as e:
        srv.submit(f, g, "y")
    assert e.value.code == rsl.RSL_ENOMEM
    srv.close()
    own.close()
