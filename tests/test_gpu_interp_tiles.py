"""GPU: the interpolation on the matrix cores at the edges of its tiles (256
coefficients), K slices (64) and segments (32), with one and with four waves per
tile, against a closed form: res_y(c y + p(x), d y + q(x)) = c q - d p.  The gapped
path (divided differences) of the same problems gives the same bits."""

import pytest

from workloads import _uniform_signed, rng_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1010_1386_amd as m
    c = m.Context(device=0, workspace_bytes=1 << 30)
    yield c
    c.close()


def problem(rng, a, b, bits):
    p, q = _uniform_signed(rng, bits, a + 1), _uniform_signed(rng, bits, b + 1)
    c, d = 7, -3
    p[a] = p[a] or 1
    q[b] = q[b] or 1
    want = [c * (q[i] if i <= b else 0) - d * (p[i] if i <= a else 0) for i in range(max(a, b) + 1)]
    while want and want[-1] == 0:
        want.pop()
    return ([p, [c] + [0] * a], [q, [d] + [0] * b], "y"), want


@pytest.mark.parametrize("D", [1, 15, 16, 31, 32, 33, 63, 64, 65, 255, 256, 257, 287, 288, 511, 512, 513, 1000, 2054,
                               3790])
def test_degree_bounds(ctx, D):
    import paper_1010_1386_amd as rsl
    rng = rng_for(960, D)
    prob, want = problem(rng, D // 2 + 1, D - D // 2, 40)  # degree bound a + b - 1
    assert rsl.query(*prob)["D"] == D
    assert ctx.res(*prob) == want
    if D <= 1000:
        assert ctx.res(*prob, interp_newton=True) == want
    assert ctx.res(*prob, point_origin=5) == want  # shifted origin after the basis change


def test_one_wave_per_tile(ctx):
    """Enough tiles for one wave each, degree bounds mixed over the tile edges."""
    import paper_1010_1386_amd as rsl
    rng = rng_for(961, 0)
    probs, want = [], []
    for k in range(150):
        D = [40, 255, 256, 300, 511, 513, 700][k % 7]
        p, w = problem(rng, D // 2 + 1, D - D // 2, 64)
        probs.append(p)
        want.append(w)
    job = ctx.job(probs)
    infos = [rsl.query(*p) for p in probs]
    assert sum(i["n_primes"] * (i["D"] // 256 + 1) for i in infos) >= 1024
    job.run("staged")
    assert job.results() == want
    job.run("plain")  # one launch per problem: four waves per tile
    assert job.results() == want
    job.close()
