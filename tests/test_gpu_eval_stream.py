"""GPU: the streamed evaluation (one lane per (prime, point), sums on the matrix
cores with one or two K slices, the lower degree in registers and the higher
one's values in LDS) gives the bits of the column layouts (Horner's rule, and
the persistent schedule) and of the oracle: both sides of every bound of its
dispatch, every remainder of the lower degree modulo 4, both orders, point
counts around a wave, points with a vanishing leading coefficient, remainders
that lose more than one degree, and common factors."""

import pytest

import oracle
from test_gpu_eval_mfma import ctx, horner, modq, rsl  # noqa: F401
from workloads import _bmul, dense_total, rng_for, small_random

pytestmark = pytest.mark.gpu


def solve(c, probs, mode="staged", **opts):
    job = c.job(probs, **opts)
    job.run(mode)
    got = job.results()
    job.close()
    return got


# (y-degree of f, x-degree of f, y-degree of g, x-degree of g)
EDGES = [(8, 31, 7, 3), (9, 32, 8, 2), (3, 63, 5, 40), (3, 64, 5, 2), (33, 4, 32, 3), (40, 3, 41, 3), (48, 2, 48, 2),
         (49, 2, 48, 2), (49, 2, 49, 2), (63, 1, 20, 2), (64, 1, 20, 2), (5, 2, 47, 3), (1, 7, 1, 9), (2, 9, 30, 1),
         (17, 33, 16, 33), (24, 34, 25, 2), (1, 2, 48, 1)]


def test_dispatch_edges(ctx, horner):  # noqa: F811
    rng = rng_for(950, 0)
    probs = [(small_random(rng, a, b, 12), small_random(rng, c, d, 12), "y") for a, b, c, d in EDGES]
    got = solve(ctx, probs)
    assert got == solve(horner, probs) == solve(ctx, probs, eval_regs=False) == solve(ctx, probs, "plain")
    modq(probs, got, 950)


@pytest.mark.parametrize("dx", [20, 33])
def test_lower_degrees_and_orders(ctx, horner, dx):  # noqa: F811
    rng = rng_for(951, dx)
    probs = []
    for n in range(1, 13):
        f, g = small_random(rng, n, dx, 20), small_random(rng, n + (n * 5) % 7, 6, 20)
        probs += [(f, g, "y"), (g, f, "y")]
    got = solve(ctx, probs)
    assert got == solve(horner, probs) == solve(ctx, probs, "batched")
    modq(probs, got, 951)


def test_point_counts_around_a_wave(ctx):  # noqa: F811
    """64, 65, 127, 128 and 129 points per prime."""
    rng = rng_for(952, 0)
    probs = [(dense_total(rng, 9, 12), dense_total(rng, 7, 12), "y")]
    want = [oracle.res(f, g, v) for f, g, v in probs]
    for extra in (0, 1, 63, 64, 65):
        assert solve(ctx, probs, extra_points=extra) == want, extra


@pytest.mark.parametrize("dx", [9, 35])
def test_leaving_the_generic_pattern(ctx, horner, dx):  # noqa: F811
    rng = rng_for(953, dx)
    r = lambda dy, d, bits=10: [list(row) for row in small_random(rng, dy, d, bits)]  # noqa: E731
    F = r(9, dx)
    F[9] = [0, -5, 1] + [0] * (dx - 2)  # lc_y = x (x - 5): points 0 and 5
    G = r(8, dx)
    G[8] = [6, -1] + [0] * (dx - 1)     # lc_y = 6 - x: point 6
    E = [row if j % 3 == 0 else [0] * (dx + 1) for j, row in enumerate(r(9, dx))]  # polynomials in y^3
    K = [row if j % 3 == 0 else [0] * (dx + 1) for j, row in enumerate(r(6, dx))]
    probs = [(F, r(9, 4), "y"), (F, G, "y"), (r(17, 3), G, "y"), (E, K, "y"), (K, E, "y"), (E, r(4, 2), "y")]
    got = solve(ctx, probs)
    assert got == solve(horner, probs) == solve(ctx, probs, "batched")
    assert solve(ctx, probs, points="formal") == got
    modq(probs, got, 953)
    h = dense_total(rng, 3, 6)  # a common factor: the resultant is zero
    assert solve(ctx, [(_bmul(h, dense_total(rng, 5, 6)), _bmul(h, dense_total(rng, 4, 6)), "y")]) == [[]]


def test_joint_pair_with_different_slices(ctx, horner):  # noqa: F811
    """The y problem (34 x-powers: two slices) writes the x problem's tiles (one slice), and back."""
    rng = rng_for(954, 0)
    for dy, dx in ((6, 33), (33, 6), (40, 45)):
        f, g = small_random(rng, dy, dx, 10), small_random(rng, dy - 1, dx - 2, 10)
        pair = [(f, g, "y"), (f, g, "x")]
        got = solve(ctx, pair)
        assert got == solve(horner, pair)
        modq(pair, got, 954)
    big = [[int(v) << 90 for v in row] for row in small_random(rng, 5, 34, 20)]  # multi-limb
    pair = [(big, small_random(rng, 6, 33, 20), "y"), (big, None, "x")]
    pair[1] = (big, pair[0][1], "x")
    assert solve(ctx, pair) == solve(horner, pair)
