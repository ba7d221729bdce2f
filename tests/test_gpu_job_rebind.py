"""GPU: a job bound to memory that only its smallest layout fits, or refused for lack
of memory, takes its usual layout again when it is bound to enough."""

import pytest

from workloads import rng_for, small_random

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsl():
    import paper_1010_1386_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(rsl):
    c = rsl.Context(device=0, workspace_bytes=1 << 28)
    yield c
    c.close()


# shapes whose digit tiles take more memory than their column layouts
@pytest.mark.parametrize("shape", [(45, 5, 11, 1), (48, 1, 40, 1), (2, 33, 3, 9)])
def test_rebind(rsl, ctx, shape):
    rng = rng_for(986, shape[0])
    a, b, c, d = shape
    f, g = small_random(rng, a, b, 30), small_random(rng, c, d, 30)
    least = rsl.query(f, g)["footprint_bytes"]
    want = ctx.res(f, g)
    job = ctx.job([(f, g, "y")])
    usual = job.info()
    roomy = usual["device_bytes"]
    assert least < roomy and usual["mulmods_sums_mfma"] > 0

    def run_all():
        for mode in ("staged", "batched", "plain"):
            job.run(mode)
            assert job.results() == [want], mode
        job.run("staged", graph=True)
        assert job.results() == [want]

    for sizes in ((least, roomy), (least, least, roomy), (least, least // 2, roomy), (roomy - 1, roomy),
                  (least // 2, roomy), (least // 2, least, roomy)):
        for size in sizes:
            if size < least:
                with pytest.raises(rsl.RSLError) as e:
                    job.bind(size)
                assert e.value.code == rsl.RSL_ENOMEM and "device bytes" in str(e.value)
                assert job.info() == usual
                with pytest.raises(rsl.RSLError):
                    job.run("staged")  # unbound
                continue
            job.bind(size)
            if size < roomy:
                assert job.info()["mulmods_sums_mfma"] == 0 and job.info()["device_bytes"] <= least
            else:
                assert job.info() == usual
            run_all()
    job.close()
