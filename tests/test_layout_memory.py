"""CPU: a job's buffers lie within its device memory, and those that are live
together do not overlap.  Random shapes and batches of them (up to degrees 63, past
them, one and many limbs, more than 512 primes), the usual layout and the one with
the least memory, chunked and whole partial sums."""

from _host_driver import run_driver

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include "job.h"
#include "stages.h"
using namespace rsl;

static std::mt19937_64 R(11);
static int pick(int lo, int hi) { return lo + static_cast<int>(R() % (hi - lo + 1)); }

struct Poly {
  std::vector<uint32_t> w;
  rsl_poly p{};
};
static Poly make(int dy, int dx, int L) {
  Poly q;
  q.w.resize(static_cast<size_t>(dy + 1) * (dx + 1) * L);
  for (uint32_t& v : q.w) v = static_cast<uint32_t>(R());
  q.p.dx = dx;
  q.p.dy = dy;
  q.p.limbs = L;
  return q;
}

struct Span {
  size_t lo, hi;
};
static bool disjoint(std::vector<Span> v) {
  std::sort(v.begin(), v.end(), [](const Span& a, const Span& b) { return a.lo < b.lo; });
  for (size_t i = 1; i < v.size(); ++i)
    if (v[i].lo < v[i - 1].hi) return false;
  return true;
}

int main() {
  int bad = 0, lean_differs = 0, wide = 0, no_digits = 0, sum = 0;
  for (int t = 0; t < 300; ++t) {
    const int n = t % 3 == 0 ? 1 : pick(1, 6);
    std::vector<Poly> ps;
    for (int k = 0; k < 2 * n; ++k) {
      const int s = t % 5, big = s == 0 ? 64 : s == 1 ? 33 : s == 2 ? 12 : s == 3 ? 5 : 80;
      const int dy = pick(1, big), dx = pick(1, std::max(1, std::min(big, 600 / dy)));
      ps.push_back(make(dy, dx, s == 3 ? pick(3, t % 2 ? 12 : 220) : 2));
    }
    std::vector<rsl_poly> f, g;
    std::vector<int> var;
    for (int k = 0; k < n; ++k) {
      for (int h = 0; h < 2; ++h) ps[2 * k + h].p.coeff = ps[2 * k + h].w.data();
      f.push_back(ps[2 * k].p);
      g.push_back(ps[2 * k + 1].p);
      var.push_back(pick(0, 1));
      if (k > 0 && pick(0, 2) == 0) {  // both projections of one system
        f[k] = f[k - 1];
        g[k] = g[k - 1];
        var[k - 1] = RSL_Y;
        var[k] = RSL_X;
      }
    }
    size_t total[2] = {};
    for (int lean = 0; lean < 2; ++lean) {
      Job J;
      J.lean = lean != 0;
      std::string err;
      const TuneConfig tc{RSL_STAGED, t % 2 ? 64 : 4096, 1, 0, t % 2, 0};
      if (job_build(nullptr, n, f.data(), g.data(), var.data(), nullptr, &J, &err, &tc)) continue;
      if (J.live.empty()) continue;
      std::vector<Span> fixed{{0, J.up_bytes}}, tiles, segs, own;
      for (size_t li = 0; li < J.live.size(); ++li) {
        const DevProblem& d = J.dev[li];
        const ProbLayout& L = J.lay[li];
        const size_t np = d.np, D1 = d.D + 1, E1 = d.E + 1;
        auto put = [](std::vector<Span>& v, size_t at, size_t bytes) { v.push_back({at, at + bytes}); };
        put(fixed, L.out, D1 * d.L_out * 4);
        put(fixed, L.zval, np * E1 * 4);
        put(fixed, L.zbad, np * E1);
        put(fixed, L.cpart, d.nchunk * np * D1 * 8);
        if (d.wide) {
          ++wide;
          put(fixed, L.wT, static_cast<size_t>(d.wdpad) * d.wnpad * 4);
          put(fixed, L.wq, D1 * 4);
          put(fixed, L.wS, D1 * 2 * d.Lw * 8);
          if (d.wide_mfma) put(fixed, L.wsum, D1 * 8);
          if (d.wide_mfma && L.crt_own) put(fixed, L.wMd, size_t(kWideDigits) * d.wlpad * d.wnpad);
        }
        put(d.evmf ? own : fixed, L.resid, np * d.CS * 4);
        if (d.evmf) put(tiles, L.dig, np * d.dfr * 512);
        put(segs, L.hseg, np * ((D1 + kCkpt - 1) / kCkpt * kCkpt) * 4);
        put(own, L.aconv, d.ncchunk * np * D1 * 8);
      }
      own.push_back({J.queue_off, J.queue_off + J.queue_bytes});
      no_digits += !J.crt_mm;
      if (!lean && !J.crt_mm) ++bad, std::printf("case %d: no digits in the usual layout\n", t);
      size_t end = 0;
      for (const std::vector<Span>* v : {&fixed, &tiles, &segs, &own}) {
        std::vector<Span> all = fixed;
        if (v != &fixed) all.insert(all.end(), v->begin(), v->end());
        if (!disjoint(all)) ++bad, std::printf("overlap %d lean %d\n", t, lean);
        for (const Span& s : *v) end = std::max(end, s.hi);
      }
      if (end > J.total)
        ++bad, std::printf("case %d lean %d: total %zu, buffers end at %zu\n", t, lean, J.total, end);
      total[lean] = J.total;
      ++sum;
    }
    lean_differs += total[1] < total[0];
  }
  std::printf("bad %d layouts %d\n", bad, sum);
  std::printf("lean differs: %d, wide: %d, no digits: %d\n", lean_differs > 0, wide > 0, no_digits > 0);
}
"""


def test_buffers(tmp_path):
    rc, out = run_driver(DRIVER, tmp_path)
    assert rc == 0, out
    lines = out.strip().split("\n")
    assert lines[-2].startswith("bad 0 layouts ") and int(lines[-2].split()[-1]) > 400, out[-2000:]
    assert lines[-1] == "lean differs: 1, wide: 1, no digits: 1"
