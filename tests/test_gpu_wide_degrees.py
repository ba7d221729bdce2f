"""GPU: resultants over more than 512 primes with degree bounds of several hundred, alone
in their call (the layouts whose partial sums would be split), twice in a row with
other work between, against the closed form res_y(c y + p, d y + q) = c q - d p."""

import pytest

from test_gpu_interp_tiles import problem
from workloads import dense_total, rng_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,bits", [(129, 16500), (300, 16500), (728, 17000), (1030, 15700)])
def test_closed_form(D, bits):
    import paper_1010_1386_amd as rsl
    rng = rng_for(989, D)
    prob, want = problem(rng, D // 2 + 1, D - D // 2, bits)
    q = rsl.query(*prob)
    assert q["D"] == D and q["n_primes"] > 512
    other = (dense_total(rng, 20, 40), dense_total(rng, 19, 40), "y")
    ctx = rsl.Context(device=0, workspace_bytes=1 << 30, table_bytes=1 << 30)
    first = ctx.res(*other)
    for opts in ({}, {"eval_lanes": 4}, {"interp_newton": True}, {"prime_start": 2}, {}):
        assert ctx.res(*prob, **opts) == want, opts
        assert ctx.res(*other) == first
    assert ctx.batch([prob, other, prob], mode="staged") == [want, first, want]
    assert ctx.batch([prob, other], mode="plain") == [want, first]
    ctx.close()
