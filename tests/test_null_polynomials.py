"""A null polynomial is refused with RSL_EINVAL.  CPU: by the planning that every
call goes through (a driver linked with the library, since the entry points need a
context).  GPU: by the entry points of one problem, which then still work."""

import ctypes

import pytest

from _host_driver import run_driver
from workloads import dense_total, rng_for

DRIVER = r"""
#include <cstdio>
#include "job.h"
int main() {
  uint32_t one[2] = {1u, 0u};
  rsl_poly p{};
  p.limbs = 2;
  p.coeff = one;
  const rsl_poly* pairs[3][2] = {{nullptr, &p}, {&p, nullptr}, {nullptr, nullptr}};
  for (auto& q : pairs) {
    rsl::Job J;
    std::string err;
    const int var = RSL_Y;
    const int rc = rsl::job_build(nullptr, 1, q[0], q[1], &var, nullptr, &J, &err);
    std::printf("%d %d %zu\n", rc, J.pstatus[0], J.live.size());
  }
}
"""


def test_planning_refuses_null(tmp_path):
    rc, out = run_driver(DRIVER, tmp_path)
    assert rc == 0
    assert out.split("\n")[:3] == ["0 -1 0"] * 3  # laid out, problem 0 refused, nothing to run


@pytest.mark.gpu
def test_entry_points_refuse_null():
    import paper_1010_1386_amd as rsl

    ctx = rsl.Context(device=0, workspace_bytes=1 << 26)
    rng = rng_for(985, 0)
    F, G = dense_total(rng, 4, 12), dense_total(rng, 3, 12)
    pf, pg = rsl.Poly(F), rsl.Poly(G)
    want = ctx.res(F, G)
    info = rsl.rsl_info()
    lib, f, g = rsl._lib, ctypes.byref(pf.c), ctypes.byref(pg.c)
    for a, b in ((None, g), (f, None), (None, None)):
        out = rsl._Result(16, 16)
        r = ctypes.byref(out.c)
        for var in (rsl.RSL_Y, rsl.RSL_X):
            assert lib.rsl_query(a, b, var, ctypes.byref(info)) == rsl.RSL_EINVAL
            assert lib.rsl_res(ctx.h, a, b, var, None, r) == rsl.RSL_EINVAL
            assert lib.rsl_res_static(ctx.h, a, b, var, None, r) == rsl.RSL_EINVAL
        assert lib.rsl_res_y(ctx.h, a, b, r) == rsl.RSL_EINVAL
        assert lib.rsl_res_x(ctx.h, a, b, r) == rsl.RSL_EINVAL
        assert lib.rsl_res_xy(ctx.h, a, b, None, r, r) == rsl.RSL_EINVAL
        assert ctx.res(F, G) == want
    ctx.close()
