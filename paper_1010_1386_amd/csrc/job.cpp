// Job layout, upload, launch and decode (see job.h).
#include "job.h"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <numeric>
#include <set>

#include "context.h"
#include "kernels.h"

namespace rsl {

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static int blocks_of(int n, int b) { return (n + b - 1) / b; }

// Algorithmic work of one (prime, point) pair: Horner multiply-adds over all
// coefficients of f and g, plus m_y n_y multiply-subtracts of the Euclidean
// remainder sequence (inversions not counted).
static int64_t pair_mulmods(const Plan& P) {
  int64_t nf = 0, ng = 0;
  for (int d : P.f.rdeg) nf += d + 1;
  for (int d : P.g.rdeg) ng += d + 1;
  return nf + ng + static_cast<int64_t>(P.my) * P.ny;
}

int job_plan(int n, const rsl_poly* f, const rsl_poly* g, const int* var, const rsl_opts* opts, Job* J,
             std::string* err) {
  J->n = n;
  J->plans.assign(n, Plan());
  J->pstatus.assign(n, 0);
  J->live.clear();
  // planning is independent per problem: spread it over host threads
  std::vector<std::string> perr(n);
  double words = 0.0;  // of the inputs, while their sizes make sense
  for (int k = 0; k < n && f && g; ++k)  // (a null polynomial is make_plan's to refuse)
    for (const rsl_poly* q : {&f[k], &g[k]})
      if (q->dx >= 0 && q->dy >= 0 && q->limbs > 0) words += (q->dx + 1.0) * (q->dy + 1.0) * q->limbs;
  parallel_for(n, host_grain(2000.0 + 8.0 * words / std::max(n, 1)), [&](int k) {
    std::string& e = perr[k];
    int rc = make_plan(&f[k], &g[k], var[k], opts, &J->plans[k], &e);
    if (!rc && !J->plans[k].zero) {
      const Plan& P = J->plans[k];
      if (P.np > kMaxPrimes) { rc = RSL_EINVAL; e = "more than 4096 primes needed (coefficients too large)"; }
      else if (P.E > 3800) { rc = RSL_EINVAL; e = "more than 3800 evaluation points needed (degree bound too large)"; }
      else if (std::max(P.my, P.ny) > 255) { rc = RSL_EINVAL; e = "degree in the eliminated variable above 255"; }
    }
    J->pstatus[k] = rc;
  });
  J->plan_err.clear();
  for (int k = 0; k < n; ++k) {
    if (J->pstatus[k]) {
      if (J->plan_err.empty()) J->plan_err = "problem " + std::to_string(k) + ": " + perr[k];
      continue;
    }
    if (!J->plans[k].zero) J->live.push_back(k);
  }
  if (err && err->empty()) *err = J->plan_err;
  return RSL_OK;
}

int64_t problem_cost(const Plan& P) {
  return pair_mulmods(P) * P.np * (P.E + 1) + static_cast<int64_t>(P.np) * (P.D + 1) * (P.D + 1);
}

int job_build(rsl_ctx* ctx, int n, const rsl_poly* f, const rsl_poly* g, const int* var, const rsl_opts* opts,
              Job* J, std::string* err, const TuneConfig* tc, bool planned, bool defer_tables) {
  if (!planned || J->n != n) job_plan(n, f, g, var, opts, J, err);
  else if (err->empty()) *err = J->plan_err;
  J->tune = tc ? *tc : TuneConfig();
  const int64_t target = std::max(64, J->tune.chunk_target);
  for (int s = 0; s < kNumStages; ++s) J->items[s].clear();
  int maxg = 0, maxE = 0, maxD = 0;
  {
    // live problems in submission order (the order below is by cost)
    std::vector<int> live;
    for (int k = 0; k < n; ++k)
      if (!J->pstatus[k] && !J->plans[k].zero) live.push_back(k);
    J->live.swap(live);
  }
  for (int k : J->live) {
    const Plan& P = J->plans[k];
    for (int gi : P.pidx) maxg = std::max(maxg, gi + 1);
    maxE = std::max(maxE, P.E);
    maxD = std::max(maxD, P.D);
  }
  // larger problems first: their work starts early and the tail is short
  std::vector<int64_t> cost(n, 0);
  for (int k : J->live) {
    const Plan& P = J->plans[k];
    cost[k] = pair_mulmods(P) * P.np * (P.E + 1);
  }
  // a system eliminated in y directly followed by the same system eliminated in
  // x shares the reduction of their common primes: the y problem writes both
  // residue tiles (pair_of[k] = the y problem of x problem k)
  std::vector<int> pair_of(n, -1);
  auto same_poly = [](const rsl_poly& a, const rsl_poly& b) {
    if (a.dx != b.dx || a.dy != b.dy || a.limbs != b.limbs) return false;
    if (a.coeff == b.coeff) return true;
    const size_t words = static_cast<size_t>(a.dx + 1) * (a.dy + 1) * a.limbs;
    return std::memcmp(a.coeff, b.coeff, words * 4) == 0;
  };
  for (int k = 1; k < n; ++k)
    if (var[k] == RSL_X && var[k - 1] == RSL_Y && !J->pstatus[k] && !J->pstatus[k - 1] &&
        !J->plans[k].zero && !J->plans[k - 1].zero && same_poly(f[k], f[k - 1]) && same_poly(g[k], g[k - 1]))
      pair_of[k] = k - 1;
  std::stable_sort(J->live.begin(), J->live.end(), [&](int a, int b) {
    // a pair ranks by its y problem, the x problem right after it
    const int ra = pair_of[a] >= 0 ? pair_of[a] : a, rb = pair_of[b] >= 0 ? pair_of[b] : b;
    if (ra == rb) return pair_of[b] >= 0 && pair_of[a] < 0;
    return cost[ra] > cost[rb] || (cost[ra] == cost[rb] && ra < rb);
  });
  J->need_g = maxg;
  J->need_E = maxE;
  J->need_D = maxD;
  if (ctx && !defer_tables && !J->live.empty()) {
    int rc = ensure_tables(ctx, maxg, maxE, maxD);
    if (rc) { *err = ctx->err; return rc; }
  }

  const int nl = static_cast<int>(J->live.size());
  J->lay.assign(nl, ProbLayout());
  J->dev.assign(nl, DevProblem());
  J->partner.assign(nl, -1);
  J->pshared.assign(nl, 0);
  J->skip_reduce.assign(nl, 0);
  {
    std::vector<int> li_of(n, -1);
    for (int li = 0; li < nl; ++li) li_of[J->live[li]] = li;
    for (int k = 0; k < n; ++k) {
      if (pair_of[k] < 0) continue;
      const int la = li_of[pair_of[k]], lb = li_of[k];
      const Plan &A = J->plans[pair_of[k]], &B = J->plans[k];
      int ns = 0;
      while (ns < A.np && ns < B.np && A.pidx[ns] == B.pidx[ns]) ++ns;
      if (ns == 0) continue;
      J->partner[la] = lb;
      J->pshared[la] = ns;
      J->skip_reduce[lb] = ns;
    }
  }
  J->pairs = 0;
  J->mulmods = 0;
  J->mm_sums_mfma = J->mm_valu = J->mfma_macs = J->interp_mm = 0;
  // stir chunking: enough blocks in flight to cover HBM latency
  int64_t stir_base = 0;
  for (int k : J->live) {
    const Plan& P = J->plans[k];
    stir_base += static_cast<int64_t>(P.np) * blocks_of(P.D + 1, 256);
  }
  // evaluation: with few (prime, point) pairs one lane per pair leaves most
  // SIMDs with a single wave; split each pair over K lanes until about four
  // waves per SIMD are in flight (problems of degree below 4K stay at one lane)
  int64_t all_pairs = 0;
  for (int k : J->live) all_pairs += static_cast<int64_t>(J->plans[k].np) * (J->plans[k].E + 1);
  int evk = J->tune.evk;
  if (opts && opts->eval_lanes > 0) evk = opts->eval_lanes;
  if (evk != 0 && evk != 1 && evk != 2 && evk != 4) {
    *err = "eval_lanes must be 0, 1, 2 or 4";
    return RSL_EINVAL;
  }
  const bool regs_ok = !(opts && opts->eval_regs < 0);
  // long_ok: shapes with |m_y - n_y| > 1 have a register form only with one
  // lane per pair (ures_regs_long)
  auto regn_of = [&](const Plan& P, bool long_ok = false) {
    if (!regs_ok || P.my < 1 || P.ny < 1 || (std::abs(P.my - P.ny) > 1 && !long_ok)) return 0;
    for (int nmax : {8, 16, 24, 32})
      if (std::max(P.my, P.ny) <= nmax) return nmax;
    return 0;
  };
  const bool evk_auto = evk <= 0;
  if (evk_auto) {
    // the register form needs no cross-lane work: keep one lane per pair for it
    bool all_regs = true;
    for (int k : J->live) all_regs = all_regs && regn_of(J->plans[k]) > 0;
    constexpr int64_t kLanesInFlight = 256LL * 4 * 4 * 64;
    evk = 1;
    if (!all_regs)
      while (evk < 4 && all_pairs * evk < kLanesInFlight) evk *= 2;
    else if (all_pairs < 2LL * 256 * 4 * 64)
      evk = 2;  // one wave can issue only about half a SIMD's rate: give each SIMD two
  }
  // the persistent schedule's partial sums laid out whole on request (one chunk)
  int dmax = 0;
  for (int k : J->live) dmax = std::max(dmax, J->plans[k].D + 1);
  const bool whole_req = (opts && opts->interp_mm > 0) || J->tune.interp_mm != 0;
  // the persistent schedule's chunk length K of the basis change, one for every
  // problem: a multiple of the checkpoint spacing, enough chunks for the target
  // number of blocks in flight
  int Kc = kCkpt;
  {
    int64_t nch = 1;
    if (stir_base < target) nch = (target + stir_base - 1) / std::max<int64_t>(stir_base, 1);
    Kc = std::max<int>(kCkpt, static_cast<int>((dmax + nch - 1) / nch));
    if (whole_req) Kc = dmax;
    Kc = (Kc + kCkpt - 1) / kCkpt * kCkpt;  // chunks start at checkpoint rows
  }
  // the streamed form (one lane per pair, sums on the matrix cores): the lower
  // degree in registers, the higher one's values in LDS
  auto stream_ok = [&](const Plan& P) {
    return regs_ok && !(ctx && ctx->eval_horner) && std::min(P.my, P.ny) >= 1 &&
           std::min(P.my, P.ny) <= kStreamDegMax && std::max(P.my, P.ny) <= kStreamLongMax &&
           P.rowf <= kMfmaXPowers && P.rowg <= kMfmaXPowers;
  };
  // Digit tiles share their memory with the buffers of the persistent schedule
  // (residue tiles, convolution sums), which the staged and plain schedules do
  // not touch.  A lean layout (for memory that the usual one does not fit) takes
  // them only within what a footprint counts for the problem in any case: those
  // buffers and its spare_bytes, the segment polynomials and, for degrees and
  // x-degrees up to 32, 2.5 KB per 16 rows and prime.  So no shape needs more than
  // its column layout and that, and a workspace sized by rsl_query runs the small
  // shapes in the streamed form (calls of degrees 8, 24 and 24 by 12: 75, 257 and
  // 140 us against 84, 302 and 176 in columns); the others' tiles can take twice
  // the column layout's memory (degrees 48 and 40, x-degree 1: 1.9 MB against 0.8).
  auto lanes_asked = [&](const Plan& P) {
    int e = 1;
    while (e < evk && std::min(P.my, P.ny) >= 4 * e * 2) e *= 2;
    return e;
  };
  auto small_shape = [&](const Plan& P) {
    const int evk_p = lanes_asked(P);
    return evk_p <= 2 && P.rowf <= 33 && P.rowg <= 33 && regn_of(P, evk_p == 1) > 0 && !(ctx && ctx->eval_horner);
  };
  auto spare_bytes = [&](const Plan& P, size_t A = 1) {
    const size_t np = P.np, rt = dig_rt(P.my + 1) + dig_rt(P.ny + 1);
    return align_up(np * align_up(static_cast<size_t>(P.D + 1), kCkpt) * 4, A) +
           (small_shape(P) ? np * rt * 2560 : 0);
  };
  // The CRT's limb digits (as many bytes as the limbs of M / p_i beside them) have
  // to fit in the same: not where a low degree needs many primes (degrees 17 and
  // 49, x-degrees 1 and 2, 219-bit coefficients: 490 primes, 0.9 MB of digits in a
  // layout of 4.4 MB).  A lean layout without them takes the column sums.
  J->crt_mm = !(ctx && ctx->crt_garner);
  if (J->crt_mm && J->lean) {
    size_t digits = 0, spare = 0;
    std::set<const CrtConst*> seen;
    for (int k : J->live) {
      const Plan& P = J->plans[k];
      spare += spare_bytes(P);
      if (seen.insert(P.crt.get()).second) digits += P.crt->dig.size();
    }
    J->crt_mm = digits <= spare;
  }
  auto tiles_fit = [&](const Plan& P, const DevProblem& d) {
    if (!J->lean) return true;
    const size_t np = P.np, rt = dig_rt(P.my + 1) + dig_rt(P.ny + 1);
    const size_t kh = (P.rowf <= 32 && P.rowg <= 32) ? 1 : 2;
    const int cchunk = (J->tune.conv_whole || whole_req) ? P.D + 1 : Kc;
    const size_t shared = np * d.CS * 4 + static_cast<size_t>(blocks_of(P.D + 1, cchunk)) * np * (P.D + 1) * 8;
    return np * rt * kh * kEvDigits * 512 + (J->crt_mm ? P.crt->dig.size() : 0) <= shared + spare_bytes(P);
  };
  J->crt_ns = 1;
  J->max_np = 0;
  J->slot_np = 0;
  J->any_schur = false;
  const bool schur_req = (opts && opts->eval_schur > 0) || J->tune.schur != 0;
  const bool newton_req = opts && opts->interp_newton > 0;
  for (int li = 0; li < nl; ++li) {
    const Plan& P = J->plans[J->live[li]];
    DevProblem& d = J->dev[li];
    d = DevProblem{};
    d.my = P.my;
    d.ny = P.ny;
    d.rowf = P.rowf;
    d.rowg = P.rowg;
    d.myp = (P.my + kRowGroup) / kRowGroup * kRowGroup;
    d.nyp = (P.ny + kRowGroup) / kRowGroup * kRowGroup;
    d.goff = P.rowf * d.myp;
    d.CS = static_cast<int>(align_up(static_cast<size_t>(d.goff) + static_cast<size_t>(P.rowg) * d.nyp, 4));
    d.ncoef = (P.my + 1) * P.rowf + (P.ny + 1) * P.rowg;
    d.L_in = std::max(P.f.L, P.g.L);
    d.D = P.D;
    d.E = P.E;
    d.origin = P.origin;
    d.formal = P.formal;
    d.np = P.np;
    d.L_out = P.L_out;
    d.kchunk = Kc;
    d.nchunk = (P.D + 1 + d.kchunk - 1) / d.kchunk;
    const bool stream = stream_ok(P) && tiles_fit(P, d);
    // with no lane count asked for, the streamed form takes every problem it
    // fits, whatever the job's size: against two lanes per pair on the
    // degree-24 pair (its smallest use) 30.2 -> 21.9 us, against the LDS columns
    // on one pair of degrees 43 and 19 154 -> 22.6 us, at degrees 42 and 41
    // 668 -> 67 us, on 64 requests of degrees 8..48 8.35 -> 0.99 ms.  The bounds
    // are the registers (lower degree 48), the LDS rows and the K slices; the
    // shapes within them were all accepted by the column layouts it replaces.
    d.evk = (evk_auto && stream) ? 1 : lanes_asked(P);
    d.evpb = 64 / d.evk;
    d.regn = (d.evk <= 2) ? regn_of(P, d.evk == 1) : 0;
    d.schur = (schur_req && P.my >= 1 && P.ny >= 1 && P.my + P.ny <= kSchurMaxR) ? 1 : 0;
    d.newton_all = newton_req ? 1 : 0;
    if (d.schur) {  // one wave per pair, kSchurPts points per block
      d.evk = 1;
      d.evpb = kSchurPts;
      d.regn = 0;
      J->any_schur = true;
    }
    // the Horner sums on the matrix cores: the streamed form, or a lane pair
    // per (prime, point) for x-degrees up to 32; one K slice of the products
    // holds x-powers 0..31, two hold 0..63
    d.evmf = (d.schur || (ctx && ctx->eval_horner)) ? 0
             : d.evk == 1 ? (stream ? 1 : 0)
                          : (d.evk == 2 && d.regn > 0 && P.rowf <= 33 && P.rowg <= 33 && tiles_fit(P, d) ? 1 : 0);
    if (d.evmf && d.evk == 1) d.regn = (std::min(P.my, P.ny) + 7) / 8 * 8;
    d.dkh = !d.evmf ? 0 : (P.rowf <= 32 && P.rowg <= 32) ? 1 : 2;
    d.dRTf = d.evmf ? dig_rt(P.my + 1) : 0;
    d.dRTg = d.evmf ? dig_rt(P.ny + 1) : 0;
    d.dfr = kEvDigits * d.dkh * (d.dRTf + d.dRTg);
    d.crt_garner = (ctx && ctx->crt_garner) ? 1 : 0;
    d.wide = P.wide ? 1 : 0;
    d.Lw = P.Lw;
    d.wide_mfma = (P.wide && !(ctx && ctx->wide_valu)) ? 1 : 0;
    d.wdpad = static_cast<int>(align_up(static_cast<size_t>(P.D + 1), kWideMfmaKT));
    d.wlpad = static_cast<int>(align_up(static_cast<size_t>(P.Lw), kWideMfmaTT));
    d.wnpad = static_cast<int>(align_up(static_cast<size_t>(P.np), kWideMfmaK));
    // the convolution's input range: the basis change's chunking, or whole
    d.cchunk = (J->tune.conv_whole || whole_req) ? P.D + 1 : d.kchunk;
    d.ncchunk = (P.D + 1 + d.cchunk - 1) / d.cchunk;
    if (!P.wide) {
      J->crt_ns = std::max(J->crt_ns, (P.np + 63) / 64);
      J->slot_np = std::max(J->slot_np, P.np);
    }
    J->max_np = std::max(J->max_np, P.np);
    J->pairs += static_cast<int64_t>(P.np) * (P.E + 1);
    J->mulmods += pair_mulmods(P) * P.np * (P.E + 1);
    {
      const int64_t pts = static_cast<int64_t>(P.np) * (P.E + 1);
      const int64_t sums = pair_mulmods(P) - static_cast<int64_t>(P.my) * P.ny;  // N_f + N_g
      if (d.evmf) {
        J->mm_sums_mfma += sums * pts;
        J->mm_valu += static_cast<int64_t>(P.my) * P.ny * pts;
        // int8 16x16x64 products per 16-point tile and 16-row tile (ev_tile_products)
        const int64_t tiles = static_cast<int64_t>(P.np) * blocks_of(P.E + 1, d.evpb) * (d.evpb / 16);
        J->mfma_macs += tiles * (d.dRTf + d.dRTg) * ev_tile_products(d.dkh) * 16 * 16 * 64;
      } else {
        J->mm_valu += pair_mulmods(P) * pts;
      }
      J->interp_mm += static_cast<int64_t>(P.np) * (P.D + 1) * (P.D + 2);
    }
  }

  if (J->crt_ns == 5 || J->crt_ns == 7) ++J->crt_ns;  // CRT kernels exist for 1-4, 6 and 8 slots per lane
  // a pair shares its reduction where both evaluate from residue tiles; digit
  // tiles are written whole by their own problem
  for (int li = 0; li < nl; ++li)
    if (J->partner[li] >= 0) {
      const int lb = J->partner[li];
      const DevProblem& b = J->dev[lb];
      DevProblem& a = J->dev[li];
      if (a.evmf || b.evmf) {
        J->partner[li] = -1;
        J->pshared[li] = J->skip_reduce[lb] = 0;
        continue;
      }
      a.pshared = J->pshared[li];
      a.pmyp = b.myp;
      a.pnyp = b.nyp;
      a.pgoff = b.goff;
      a.pCS = b.CS;
    }

  // work items, problem by problem (so that each problem's items are
  // contiguous): each problem's items of each stage are counted, the lists
  // sized, and every problem writes its own ranges (in parallel)
  auto emit = [&](int li, int s, WorkItem* out) -> int {
    const Plan& P = J->plans[J->live[li]];
    const DevProblem& d = J->dev[li];
    int c = 0;
    // blocks 0..nb-1 of every step-th slot of s0..np-1
    auto put = [&](int s0, int np, int step, int nb, int sub) {
      if (out)
        for (int sl = s0; sl < np; sl += step)
          for (int b = 0; b < nb; ++b) out[c++] = WorkItem{li, sl, b, sub};
      else if (s0 < np)
        c += (np - s0 + step - 1) / step * nb;
    };
    switch (s) {
      case kStageReduce: {
        // slots below skip_reduce are reduced by the partner (the same system
        // in y); item slot 0 of block 0 also clears the statuses, so a problem
        // whose slots are all shared keeps one such item
        const int s0 = J->skip_reduce[li];
        if (d.evmf) {
          const int spw = d.L_in <= 2 ? kReduceSlotsShort : kReduceSlotsLong;
          put(0, P.np, 4 * spw, reduce_tile_blocks(d), spw);
        } else if (d.L_in > 2) {  // long limb chains: staged limbs, eight primes per thread
          const int first = (s0 / kReduceMlSlots) * kReduceMlSlots;
          put(first, P.np, kReduceMlSlots, blocks_of(d.CS, kReduceMlCoeffs), 1);
          if (first > 0) put(0, 1, 1, 1, 1);
        } else {
          put(s0, P.np, 1, blocks_of(d.CS, 256), 0);
          if (s0 > 0) put(0, 1, 1, 1, 0);
        }
        break;
      }
      case kStageEval:
        put(0, P.np, 1, blocks_of(P.E + 1, d.evpb), 0);
        break;
      case kStageConv:  // Newton coefficients and segment polynomials, then the basis change:
      case kStageStir:  // tiles of 256 coefficients
        put(0, P.np, 1, blocks_of(P.D + 1, kTile), 0);
        break;
      case kStageNewton:
        // gapped interpolation is possible only with a non-constant leading
        // coefficient (bad points) or a shifted origin
        if (P.origin != 0 || (!P.formal && P.s > 0) || d.newton_all) put(0, P.np, 1, 1, 0);
        break;
      case kStageCrt:
        if (!P.wide) put(-1, 0, 1, blocks_of(P.D + 1, J->crt_mm ? kCrtMmRows : kCrtWaves), 0);
        break;
    }
    return c;
  };
  {
    constexpr int kLists = kNumStages;
    std::vector<int>& cnt = J->tmp_a;
    cnt.assign(static_cast<size_t>(nl) * kLists, 0);
    for (int li = 0; li < nl; ++li)
      for (int s = 0; s < kLists; ++s) cnt[static_cast<size_t>(li) * kLists + s] = emit(li, s, nullptr);
    std::vector<int>& off = J->tmp_b;
    off.assign(cnt.size(), 0);
    // the evaluation items grouped by layout variant and the reduce items by kind
    // (problem order within one): each is one launch of the staged schedule
    std::vector<int>& var_of = J->tmp_c;
    var_of.resize(nl);
    int nv = 1;
    for (int li = 0; li < nl; ++li) {
      var_of[li] = eval_variant(J->dev[li]);
      nv = std::max(nv, var_of[li] + 1);
    }
    auto kind_of = [&](int li) { return !J->dev[li].evmf ? 0 : J->dev[li].L_in <= 2 ? 1 : 2; };
    J->eval_vstart.assign(static_cast<size_t>(nv) + 1, 0);
    for (int s = 0; s < kLists; ++s) {
      int o = 0;
      for (int v = 0; v < (s == kStageEval ? nv : s == kStageReduce ? 3 : 1); ++v) {
        if (s == kStageEval) J->eval_vstart[v] = o;
        if (s == kStageReduce) J->reduce_start[v] = o;
        for (int li = 0; li < nl; ++li) {
          if (s == kStageEval && var_of[li] != v) continue;
          if (s == kStageReduce && kind_of(li) != v) continue;
          off[static_cast<size_t>(li) * kLists + s] = o;
          o += cnt[static_cast<size_t>(li) * kLists + s];
        }
      }
      if (s == kStageEval) J->eval_vstart[nv] = o;
      if (s == kStageReduce) J->reduce_start[3] = o;
      J->items[s].clear();
      J->items[s].resize(o);
    }
    double total = 0.0;
    for (int s = 0; s < kLists; ++s) total += J->items[s].size();
    parallel_for(nl, host_grain(50.0 + 3.0 * total / std::max(nl, 1)), [&](int li) {
      ProbLayout& L = J->lay[li];
      for (int s = 0; s < kLists; ++s) {
        const size_t at = static_cast<size_t>(li) * kLists + s;
        emit(li, s, J->items[s].data() + off[at]);
        L.item_begin[s] = off[at];
        L.item_end[s] = off[at] + cnt[at];
      }
    });
  }

  // wide CRT items, problem by problem
  for (int pass = 0; pass < 3; ++pass) J->wide_items[pass].clear();
  J->wide_mfma = false;
  J->wdig_items.clear();
  J->wdig_lds = 0;
  for (int li = 0; li < nl; ++li) {
    const Plan& P = J->plans[J->live[li]];
    const DevProblem& d = J->dev[li];
    ProbLayout& L = J->lay[li];
    for (int pass = 0; pass < 3; ++pass) L.wide_begin[pass] = static_cast<int>(J->wide_items[pass].size());
    if (P.wide) {
      for (int b = 0; b < blocks_of(P.D + 1, kWideTCoeffs); ++b) J->wide_items[0].push_back({li, -1, b, 0});
      // column sums: the blocks of one limb tile read the same columns of
      // the M_i table, so they are dealt onto one XCD (workgroup i of a launch
      // runs on XCD i mod 8; a problem's range starts anywhere, but its items
      // of one tile keep one residue mod 8)
      constexpr int kXcds = 8;
      const bool mfma = d.wide_mfma != 0;
      J->wide_mfma = mfma;
      const int nkt = mfma ? d.wdpad / kWideMfmaKT : blocks_of(P.D + 1, kWideKT);
      const int nht = mfma ? d.wlpad / kWideMfmaTT : blocks_of(P.Lw, kWideHT);
      std::vector<std::vector<WorkItem>> bins(kXcds);
      for (int ht = 0; ht < nht; ++ht)
        for (int kt = 0; kt < nkt; ++kt) bins[ht % kXcds].push_back({li, -1, kt, ht});
      std::vector<size_t> pos(kXcds, 0);
      for (int t = 0; t < nkt * nht; ++t) {
        int x = t % kXcds;
        if (pos[x] >= bins[x].size()) {  // bin x is empty: take from the fullest
          size_t best = 0;
          for (int y = 0; y < kXcds; ++y)
            if (bins[y].size() - pos[y] > best) {
              best = bins[y].size() - pos[y];
              x = y;
            }
        }
        J->wide_items[1].push_back(bins[x][pos[x]++]);
      }
      for (int k = 0; k <= P.D; ++k) J->wide_items[2].push_back({li, -1, k, 0});
    }
    for (int pass = 0; pass < 3; ++pass) L.wide_end[pass] = static_cast<int>(J->wide_items[pass].size());
  }

  // evaluation items: grouped by layout variant as they were written (a
  // problem's items stay together, as the one-pipeline-per-problem schedule needs)
  {
    const std::vector<WorkItem>& ev = J->items[kStageEval];
    const std::vector<int>& vstart = J->eval_vstart;
    const int nv = static_cast<int>(vstart.size()) - 1;
    J->eval_ranges.clear();
    // each variant's launch sized for its own problems (a small register
    // form keeps more waves per CU than the largest problem's LDS would allow)
    std::vector<size_t> vlds(static_cast<size_t>(nv), 0);
    for (int li = 0; li < nl; ++li)
      vlds[J->tmp_c[li]] = std::max(vlds[J->tmp_c[li]], static_cast<size_t>(eval_stage_lds_words(J->dev[li])) * 4);
    for (int v = 0; v < nv; ++v)
      if (vstart[v] < vstart[v + 1])
        J->eval_ranges.push_back({v, static_cast<int>(vstart[v]), static_cast<int>(vstart[v + 1]), vlds[v]});
    // the staged launches take the same items dealt so that all blocks of one
    // (problem, prime) run on the same XCD: workgroup i of a launch goes to
    // XCD i mod 8, so the prime's coefficient tile is fetched into one L2
    // instead of eight.  Per variant range: the g-th (problem, prime) of the
    // range goes to bin g mod 8, and launch position t takes the next item of
    // bin t mod 8 (of the bin with the most items left once that one is empty).
    // Each bin is a cursor over the range's problems, so an item costs a few
    // instructions and no memory but its own; the ranges are independent.
    constexpr int kXcds = 8;
    J->eval_staged.resize(ev.size());
    parallel_for(static_cast<int>(J->eval_ranges.size()), host_grain(4.0 * ev.size() / std::max<size_t>(1, J->eval_ranges.size())),
                 [&](int ri) {
      const auto& R = J->eval_ranges[ri];
      struct Bin {
        int li, slot, blk, nb, np;  // the next item; blocks and primes of its problem
        int64_t left;               // items of the bin
      } bin[kXcds] = {};
      auto settle = [&](Bin& B) {  // slots past a problem's end are the next problem's
        while (B.li < nl && (J->tmp_c[B.li] != R.variant || B.slot >= J->dev[B.li].np)) {
          if (J->tmp_c[B.li] == R.variant) B.slot -= J->dev[B.li].np;
          ++B.li;
        }
        if (B.li < nl) {
          B.np = J->dev[B.li].np;
          B.nb = blocks_of(J->dev[B.li].E + 1, J->dev[B.li].evpb);
        }
      };
      int g = 0;  // (problem, prime) groups before this problem, mod 8
      for (int li = 0; li < nl; ++li) {
        if (J->tmp_c[li] != R.variant) continue;
        const int np = J->dev[li].np, nb = blocks_of(J->dev[li].E + 1, J->dev[li].evpb);
        for (int x = 0; x < kXcds; ++x)
          bin[x].left += static_cast<int64_t>((np + 7 - (x - g + kXcds) % kXcds) / kXcds) * nb;
        g = (g + np) % kXcds;
      }
      for (int x = 0; x < kXcds; ++x) {
        bin[x].slot = x;
        settle(bin[x]);
      }
      WorkItem* out = J->eval_staged.data() + R.begin;
      const int total = R.end - R.begin;
      for (int t = 0; t < total; ++t) {
        int x = t % kXcds;
        if (bin[x].left == 0) {  // bin x is empty: take from the fullest
          int64_t best = 0;
          for (int y = 0; y < kXcds; ++y)
            if (bin[y].left > best) {
              best = bin[y].left;
              x = y;
            }
        }
        Bin& B = bin[x];
        --B.left;
        out[t] = WorkItem{B.li, B.slot, B.blk, 0};
        if (++B.blk == B.nb) {
          B.blk = 0;
          B.slot += kXcds;
          if (B.slot >= B.np) settle(B);
        }
      }
    });
  }

  // device layout: [problems | items | inputs | statuses][outputs][intermediates]
  const size_t A = 256;
  size_t o = 0;
  J->probs_off = o;
  o = align_up(o + sizeof(DevProblem) * std::max(nl, 1), A);
  for (int s = 0; s < kNumStages; ++s) {
    J->items_off[s] = o;
    o = align_up(o + sizeof(WorkItem) * J->items[s].size(), A);
  }
  J->evs_off = o;
  o = align_up(o + sizeof(WorkItem) * J->eval_staged.size(), A);
  for (int pass = 0; pass < 3; ++pass) {
    J->wide_off[pass] = o;
    o = align_up(o + sizeof(WorkItem) * J->wide_items[pass].size(), A);
  }
  // CRT constants are laid out once per prime list (problems with the same
  // canonical list share them); the wide path's digit planes are built on the
  // device by the owning problem's items
  {
    std::map<const CrtConst*, int> crt_owner;
    for (int li = 0; li < nl; ++li) {
      const Plan& P = J->plans[J->live[li]];
      const DevProblem& d = J->dev[li];
      ProbLayout& L = J->lay[li];
      const auto own = crt_owner.emplace(P.crt.get(), li);
      L.crt_own = own.second;
      L.crt_from = own.first->second;
      if (L.crt_own && d.wide_mfma) {
        J->wdig_lds = std::max(J->wdig_lds, static_cast<size_t>(wide_digits_lds_words(d)) * 4);
        for (int b = 0; b < d.wnpad / kWideMfmaK; ++b)
          for (int t = 0; t < blocks_of(d.wlpad, kWideDigitLimbs); ++t) J->wdig_items.push_back({li, -1, b, t});
      }
    }
  }
  J->wdig_off = o;
  o = align_up(o + sizeof(WorkItem) * J->wdig_items.size(), A);
  size_t digit_bytes = 0, spared_bytes = 0;
  for (int li = 0; li < nl; ++li) {
    const Plan& P = J->plans[J->live[li]];
    const DevProblem& d = J->dev[li];
    ProbLayout& L = J->lay[li];
    L.L_in = d.L_in;
    L.coeff = o; o = align_up(o + static_cast<size_t>(d.ncoef) * d.L_in * 4, 16);
    L.gdeg = o;  o = align_up(o + static_cast<size_t>(d.myp + d.nyp) / kRowGroup * 4, 16);
    L.pidx = o;  o = align_up(o + static_cast<size_t>(P.np) * 4, 16);
    if (!L.crt_own) {
      const ProbLayout& S = J->lay[L.crt_from];
      L.Hm = S.Hm; L.NH = S.NH; L.Mi = S.Mi; L.Mdig = S.Mdig; L.wdir = S.wdir; L.rinv = S.rinv; L.negM = S.negM;
      L.Mw = S.Mw; L.NHM = S.NHM; L.Tg = S.Tg; L.invM = S.invM; L.Plimb = S.Plimb;
      continue;
    }
    L.Hm = o;    o = align_up(o + static_cast<size_t>(P.np) * 4, 16);
    L.NH = o;    o = align_up(o + static_cast<size_t>(P.L_out) * 4, 16);
    // (the wide path's matrix products take the M_i from M itself)
    L.Mi = o;
    (d.wide_mfma ? spared_bytes : o) += align_up(static_cast<size_t>(P.np) * P.Lw * 4, 16);
    L.Mdig = o;
    if (J->crt_mm) {
      o = align_up(o + P.crt->dig.size(), 16);
      digit_bytes += P.crt->dig.size();
    }
    L.wdir = o;  o = align_up(o + static_cast<size_t>(P.np) * 4, 16);
    L.rinv = o;  o = align_up(o + static_cast<size_t>(P.np) * 8, 16);
    L.negM = o;  o = align_up(o + static_cast<size_t>(P.Lw) * 4, 16);
    L.Mw = L.NHM = 0;
    if (P.wide) {
      L.Mw = o;  o = align_up(o + static_cast<size_t>(P.Lw) * 4, 16);
      L.NHM = o; o = align_up(o + static_cast<size_t>(P.L_out) * 4, 16);
    }
    if (!P.canonical) {
      L.Tg = o;    o = align_up(o + static_cast<size_t>(P.np) * P.np * 4, 16);
      L.invM = o;  o = align_up(o + static_cast<size_t>(P.np) * 4, 16);
      L.Plimb = o; o = align_up(o + static_cast<size_t>(P.np) * P.L_out * 4, 16);
    }
  }
  // persistent queue: [state | tasks | ready | counters]; an initial image is
  // uploaded with the inputs and copied to the live queue before each launch
  {
    int64_t cap = 0, crt_total = 0, initial = 0;
    for (int li = 0; li < nl; ++li) {
      const Plan& P = J->plans[J->live[li]];
      const DevProblem& d = J->dev[li];
      const int64_t ne = blocks_of(P.E + 1, d.evpb), nc = blocks_of(P.D + 1, 64);
      const int64_t ns = blocks_of(P.D + 1, 64) * d.nchunk;
      cap += static_cast<int64_t>(P.np) * (1 + ne + std::max<int64_t>(nc * d.ncchunk + ns + (P.origin != 0), 1));
      const int64_t ncrt = blocks_of(P.D + 1, kCrtPerTask);
      cap += ncrt;
      crt_total += ncrt;
      initial += P.np;
    }
    J->q_capacity = static_cast<int>(std::max<int64_t>(cap, 1));
    J->q_crt_total = static_cast<int>(crt_total);
    J->q_initial = static_cast<int>(initial);
    size_t qo = 0;
    qo = align_up(qo + sizeof(QueueState), A);
    J->q_tasks = qo;
    qo = align_up(qo + sizeof(Task) * J->q_capacity, A);
    J->q_ready = qo;
    qo = align_up(qo + sizeof(int) * J->q_capacity, A);
    J->q_counters = qo;
    qo = align_up(qo + sizeof(ProbCounters) * std::max(nl, 1), A);
    J->queue_bytes = qo;
    o = align_up(o, A);
    J->qinit_off = o;
    o += J->queue_bytes;
  }
  o = align_up(o, A);
  J->status_off = o;
  for (int li = 0; li < nl; ++li) {
    J->lay[li].status = o;
    o += static_cast<size_t>(2 * J->plans[J->live[li]].np + 2) * 4;
  }
  o = align_up(o, A);
  J->status_bytes = o - J->status_off;
  J->up_bytes = o;
  J->down_off = J->status_off;
  for (int li = 0; li < nl; ++li) {
    const Plan& P = J->plans[J->live[li]];
    J->lay[li].out = o;
    o = align_up(o + static_cast<size_t>(P.D + 1) * P.L_out * 4, 16);
  }
  o = align_up(o, A);
  J->down_bytes = o - J->down_off;
  for (int li = 0; li < nl; ++li) {
    const Plan& P = J->plans[J->live[li]];
    const DevProblem& d = J->dev[li];
    ProbLayout& L = J->lay[li];
    const size_t np = P.np;
    if (!d.evmf) {
      L.resid = o;
      o = align_up(o + np * d.CS * 4, A);
    }
    L.zval = o;  o = align_up(o + np * (P.E + 1) * 4, A);
    L.zbad = o;  o = align_up(o + np * (P.E + 1), A);
    L.cpart = o; o = align_up(o + static_cast<size_t>(d.nchunk) * np * (P.D + 1) * 8, A);
    L.wT = L.wq = L.wS = L.wMd = L.wsum = 0;
    if (P.wide) {
      if (!L.crt_own) {
        L.wMd = J->lay[L.crt_from].wMd;  // the owner comes first
      } else if (d.wide_mfma) {
        L.wMd = o; o = align_up(o + static_cast<size_t>(kWideDigits) * d.wlpad * d.wnpad, A);
        spared_bytes += static_cast<size_t>(d.wlpad) * d.wnpad;
      }
      L.wT = o; o = align_up(o + static_cast<size_t>(d.wdpad) * d.wnpad * 4, A);
      L.wq = o; o = align_up(o + static_cast<size_t>(P.D + 1) * 4, A);
      L.wS = o; o = align_up(o + static_cast<size_t>(P.D + 1) * 2 * P.Lw * 8, A);
      if (d.wide_mfma) {
        L.wsum = o;
        o = align_up(o + static_cast<size_t>(P.D + 1) * 8, A);
        digit_bytes += align_up(static_cast<size_t>(P.D + 1) * 8, A);
      }
    }
  }
  // one region for buffers that are never live together: the digit tiles of the
  // staged and plain schedules (read by the evaluation), their segment
  // polynomials (interpolation only), and the persistent schedule's residue tiles
  // (of problems with digit tiles), convolution sums and live queue.  Each is
  // written before it is read, in every run.  The footprint counts them side by
  // side (the tiles as spare_bytes does) with the M_i and without the digits that
  // the image has or spares, and is at least what they take: a measure of a problem
  // that stays the same for budgets and workspaces -- what one refused stays
  // refused -- and of which the layouts touch 0.88 on average (1500 random shapes,
  // 0.54 at least).
  {
    size_t tiles = o, segs = o, own = o, apart = o;
    for (int li = 0; li < nl; ++li) {
      const Plan& P = J->plans[J->live[li]];
      const DevProblem& d = J->dev[li];
      ProbLayout& L = J->lay[li];
      const size_t np = P.np;
      L.dig = 0;
      if (d.evmf) {
        L.dig = tiles;
        tiles = align_up(tiles + np * d.dfr * 512, A);
        L.resid = own;
        own = align_up(own + np * d.CS * 4, A);
      }
      L.hseg = segs;
      segs = align_up(segs + np * align_up(static_cast<size_t>(P.D + 1), kCkpt) * 4, A);
      L.aconv = own;
      own = align_up(own + static_cast<size_t>(d.ncchunk) * np * (P.D + 1) * 8, A);
      apart += spare_bytes(P, A);
    }
    J->queue_off = own;
    own = align_up(own + J->queue_bytes, A);
    const size_t counted = own + (apart - o) + spared_bytes;
    o = std::max({tiles, segs, own, counted > digit_bytes ? counted - digit_bytes : 0});
  }
  J->total = o;

  // LDS per stage launch (max over problems)
  for (int s = 0; s < kNumStages; ++s) J->stage_lds[s] = 0;
  for (int li = 0; li < nl; ++li) {
    const DevProblem& d = J->dev[li];
    auto up = [&](int s, size_t words) { J->stage_lds[s] = std::max(J->stage_lds[s], words * 4); };
    up(kStageEval, eval_stage_lds_words(d));
    up(kStageConv, interp_coeffs_lds_words(d.D, 4));
    up(kStageStir, interp_basis_lds_words(4));
    if (J->lay[li].item_end[kStageNewton] > J->lay[li].item_begin[kStageNewton]) up(kStageNewton, newton_lds_words(d, 1024));
    if (!d.wide)
      up(kStageCrt, J->crt_mm ? crt_mm_lds_words(d.np, 4) : crt_lds_words(d, J->crt_ns, crt_block_waves(J->crt_ns)));
    if (d.L_in > 2 && !d.evmf) up(kStageReduce, reduce_ml_lds_words());
  }
  for (int pass = 0; pass < 3; ++pass) J->wide_lds[pass] = 0;
  for (int li = 0; li < nl; ++li) {
    const DevProblem& d = J->dev[li];
    if (!d.wide) continue;
    J->wide_lds[0] = static_cast<size_t>(wide_t_lds_words()) * 4;
    J->wide_lds[1] = static_cast<size_t>(J->wide_mfma ? wide_mfma_lds_words() : wide_sum_lds_words()) * 4;
    J->wide_lds[2] = std::max(J->wide_lds[2], static_cast<size_t>(wide_fin_lds_words(d)) * 4);
  }
  J->persist_lds = 0;
  for (int li = 0; li < nl; ++li) {
    const DevProblem& d = J->dev[li];
    size_t w = std::max(eval_group_lds_words(d, d.evk), eval_lds_words(d));  // no register form here
    w = std::max<size_t>(w, static_cast<size_t>(std::min(d.cchunk, d.D + 1)) + std::min(d.D + 1, d.cchunk + 64));
    w = std::max<size_t>(w, basis_lds_words(64, d.kchunk));
    if (J->lay[li].item_end[kStageNewton] > J->lay[li].item_begin[kStageNewton])
      w = std::max<size_t>(w, newton_lds_words(d, 64));
    if (!d.wide) w = std::max<size_t>(w, crt_lds_words(d, J->crt_ns, 1));
    J->persist_lds = std::max(J->persist_lds, w * 4);
  }
  for (int s = 0; s < kNumStages; ++s)
    if (J->stage_lds[s] > static_cast<size_t>(kLdsWords) * 4 ||
        (s < 3 && J->wide_lds[s] > static_cast<size_t>(kLdsWords) * 4)) {
      *err = "a stage needs more than 64 KB of LDS";
      return RSL_EINVAL;
    }
  return RSL_OK;
}

void job_bind(Job* J, uint8_t* base, uint8_t* image, bool with_queue) {
  J->base = base;
  J->with_queue = with_queue;
  const int nl = static_cast<int>(J->live.size());
  if (!image) {
    J->blob.assign(J->up_bytes, 0);
    image = J->blob.data();
  } else {
    J->blob.clear();
    // an external image is not zeroed: the queue's ready flags and the
    // statuses must start at zero (every other region is written whole)
    if (with_queue) std::memset(image + J->qinit_off, 0, J->up_bytes - J->qinit_off);
  }
  J->image = image;
  uint8_t* blob = image;
  // each problem writes its own regions (a shared CRT block only by its owner)
  double words = 0.0;
  for (int li = 0; li < nl; ++li) words += static_cast<double>(J->dev[li].ncoef) * J->lay[li].L_in;
  parallel_for(nl, host_grain(300.0 + 2.0 * words / std::max(nl, 1)), [&](int li) {
    const Plan& P = J->plans[J->live[li]];
    const ProbLayout& L = J->lay[li];
    DevProblem& d = J->dev[li];
    // inputs: f rows 0..my (stride rowf) then g rows 0..ny (stride rowg),
    // sign-extended to L_in limbs
    uint32_t* c = reinterpret_cast<uint32_t*>(blob + L.coeff);
    const int Li = L.L_in;
    auto put = [&](const View& V, int rows, int rowstride, size_t first) {
      for (int j = 0; j < rows; ++j)
        for (int i = 0; i < rowstride; ++i) {
          uint32_t* dst = c + (first + static_cast<size_t>(j) * rowstride + i) * Li;
          if (i <= V.rdeg[j]) {
            const uint32_t* src = &V.c[(static_cast<size_t>(j) * (V.dx + 1) + i) * V.L];
            const uint32_t ext = (src[V.L - 1] >> 31) ? 0xFFFFFFFFu : 0u;
            for (int l = 0; l < Li; ++l) dst[l] = (l < V.L) ? src[l] : ext;
          } else {
            for (int l = 0; l < Li; ++l) dst[l] = 0;
          }
        }
    };
    put(P.f, P.my + 1, P.rowf, 0);
    put(P.g, P.ny + 1, P.rowg, static_cast<size_t>(P.my + 1) * P.rowf);
    int* gd = reinterpret_cast<int*>(blob + L.gdeg);
    const int gf = d.myp / kRowGroup, gg = d.nyp / kRowGroup;
    for (int q = 0; q < gf; ++q) {
      int m = -1;
      for (int j = q * kRowGroup; j < (q + 1) * kRowGroup && j <= P.my; ++j) m = std::max(m, P.f.rdeg[j]);
      gd[q] = m;
    }
    for (int q = 0; q < gg; ++q) {
      int m = -1;
      for (int j = q * kRowGroup; j < (q + 1) * kRowGroup && j <= P.ny; ++j) m = std::max(m, P.g.rdeg[j]);
      gd[gf + q] = m;
    }
    std::memcpy(blob + L.pidx, P.pidx.data(), P.np * 4);
    if (L.crt_own) {
    std::memcpy(blob + L.Hm, P.crt->Hm.data(), P.np * 4);
    std::memcpy(blob + L.NH, P.crt->NH.data(), P.L_out * 4);
    if (!d.wide_mfma) std::memcpy(blob + L.Mi, P.crt->Mi.data(), P.crt->Mi.size() * 4);
    if (J->crt_mm && !P.crt->dig.empty()) std::memcpy(blob + L.Mdig, P.crt->dig.data(), P.crt->dig.size());
    std::memcpy(blob + L.wdir, P.crt->wdir.data(), P.crt->wdir.size() * 4);
    std::memcpy(blob + L.rinv, P.crt->rinv.data(), P.crt->rinv.size() * 4);
    std::memcpy(blob + L.negM, P.crt->negM.data(), P.crt->negM.size() * 4);
    if (P.wide) {
      std::memcpy(blob + L.Mw, P.crt->Mw.data(), P.crt->Mw.size() * 4);
      std::memcpy(blob + L.NHM, P.crt->NHM.data(), P.crt->NHM.size() * 4);
    }
    if (!P.canonical) {
      std::memcpy(blob + L.Tg, P.crt->Tg.data(), P.crt->Tg.size() * 4);
      std::memcpy(blob + L.invM, P.crt->invM.data(), P.crt->invM.size() * 4);
      std::memcpy(blob + L.Plimb, P.crt->Plimb.data(), P.crt->Plimb.size() * 4);
    }
    }  // crt_own
    // device pointers
    d.coeff = reinterpret_cast<const uint32_t*>(base + L.coeff);
    d.gdeg = reinterpret_cast<const int*>(base + L.gdeg);
    d.pidx = reinterpret_cast<const int*>(base + L.pidx);
    d.Hm = reinterpret_cast<const uint32_t*>(base + L.Hm);
    d.NH = reinterpret_cast<const uint32_t*>(base + L.NH);
    d.Mi = d.wide_mfma ? nullptr : reinterpret_cast<const uint32_t*>(base + L.Mi);
    d.Mdig = J->crt_mm ? base + L.Mdig : nullptr;
    d.wdir = reinterpret_cast<const uint32_t*>(base + L.wdir);
    d.rinv = reinterpret_cast<const uint32_t*>(base + L.rinv);
    d.negM = reinterpret_cast<const uint32_t*>(base + L.negM);
    d.Mw = P.wide ? reinterpret_cast<const uint32_t*>(base + L.Mw) : nullptr;
    d.NHM = P.wide ? reinterpret_cast<const uint32_t*>(base + L.NHM) : nullptr;
    d.wT = P.wide ? reinterpret_cast<uint32_t*>(base + L.wT) : nullptr;
    d.wq = P.wide ? reinterpret_cast<uint32_t*>(base + L.wq) : nullptr;
    d.wS = P.wide ? reinterpret_cast<uint64_t*>(base + L.wS) : nullptr;
    d.wsum = (P.wide && d.wide_mfma) ? reinterpret_cast<uint64_t*>(base + L.wsum) : nullptr;
    d.wMd = (P.wide && d.wide_mfma) ? reinterpret_cast<int8_t*>(base + L.wMd) : nullptr;
    d.resid = reinterpret_cast<uint32_t*>(base + L.resid);
    d.dig = d.evmf ? reinterpret_cast<uint64_t*>(base + L.dig) : nullptr;
    d.zval = reinterpret_cast<uint32_t*>(base + L.zval);
    d.zbad = base + L.zbad;
    d.aconv = reinterpret_cast<uint64_t*>(base + L.aconv);
    d.cpart = reinterpret_cast<uint64_t*>(base + L.cpart);
    d.hseg = reinterpret_cast<uint32_t*>(base + L.hseg);
    d.hstride = static_cast<int>(align_up(static_cast<size_t>(P.D + 1), kCkpt));
    d.out = reinterpret_cast<uint32_t*>(base + L.out);
    d.status = reinterpret_cast<int*>(base + L.status);
  });
  for (int li = 0; li < nl; ++li) {
    const int pa = J->partner[li];
    J->dev[li].presid = (pa >= 0) ? reinterpret_cast<uint32_t*>(base + J->lay[pa].resid) : nullptr;
  }
  // initial queue image: one REDUCE task per (problem, prime slot), largest problems first
  // (none when a problem has more primes than the persistent schedule takes)
  if (with_queue && J->max_np <= kMaxSlots) {
    uint8_t* q = blob + J->qinit_off;
    QueueState* qs = reinterpret_cast<QueueState*>(q);
    Task* tasks = reinterpret_cast<Task*>(q + J->q_tasks);
    int* ready = reinterpret_cast<int*>(q + J->q_ready);
    ProbCounters* cnt = reinterpret_cast<ProbCounters*>(q + J->q_counters);
    int t = 0;
    for (int li = 0; li < nl; ++li) {
      const Plan& P = J->plans[J->live[li]];
      const DevProblem& d = J->dev[li];
      const int ne = blocks_of(P.E + 1, d.evpb), nc = blocks_of(P.D + 1, 64);
      cnt[li].slots_left = P.np;
      for (int sl = 0; sl < P.np; ++sl) {
        cnt[li].eval_left[sl] = ne;
        cnt[li].conv_left[sl] = nc * d.ncchunk;
        cnt[li].stir_left[sl] = nc * d.nchunk;
        tasks[t] = Task{(kTaskReduce << 24) | li, sl, 0, 0};
        ready[t] = 1;
        ++t;
      }
    }
    qs->head = 0;
    qs->tail = t;
    qs->done = (J->q_crt_total == 0) ? 1 : 0;
    qs->crt_done = 0;
    qs->err = 0;
  }
  std::memcpy(blob + J->probs_off, J->dev.data(), sizeof(DevProblem) * nl);
  for (int s = 0; s < kNumStages; ++s)
    if (!J->items[s].empty())
      std::memcpy(blob + J->items_off[s], J->items[s].data(), sizeof(WorkItem) * J->items[s].size());
  if (!J->eval_staged.empty())
    std::memcpy(blob + J->evs_off, J->eval_staged.data(), sizeof(WorkItem) * J->eval_staged.size());
  for (int pass = 0; pass < 3; ++pass)
    if (!J->wide_items[pass].empty())
      std::memcpy(blob + J->wide_off[pass], J->wide_items[pass].data(), sizeof(WorkItem) * J->wide_items[pass].size());
  if (!J->wdig_items.empty())
    std::memcpy(blob + J->wdig_off, J->wdig_items.data(), sizeof(WorkItem) * J->wdig_items.size());
}

// CRT tables: canonical prime lists use the context's global tables.
static void bind_crt_tables(const rsl_ctx* ctx, Job* J) {
  const int nl = static_cast<int>(J->live.size());
  for (int li = 0; li < nl; ++li) {
    const Plan& P = J->plans[J->live[li]];
    const ProbLayout& L = J->lay[li];
    DevProblem& d = J->dev[li];
    if (P.canonical) {
      d.Tg = ctx->d_Tg;
      d.tgs = ctx->garner_np;
      d.invM = ctx->d_invM;
      d.Plimb = ctx->d_Plimb;
      d.LP = ctx->LPg;
    } else {
      d.Tg = reinterpret_cast<const uint32_t*>(J->base + L.Tg);
      d.tgs = P.np;
      d.invM = reinterpret_cast<const uint32_t*>(J->base + L.invM);
      d.Plimb = reinterpret_cast<const uint32_t*>(J->base + L.Plimb);
      d.LP = P.L_out;
    }
  }
  std::memcpy(J->image + J->probs_off, J->dev.data(), sizeof(DevProblem) * nl);
}

int job_upload_copy(rsl_ctx* ctx, Job* J, hipStream_t st, uint8_t* pinned) {
  bind_crt_tables(ctx, J);
  const size_t up = upload_bytes(*J);
  if (up == 0) return RSL_OK;
  if ((J->blob.empty() && J->image) || J->direct_image) {
    pinned = J->image;  // bound straight into pinned staging, or sent from pageable memory
  } else {
    if (!pinned) {
      int rc = ensure_staging(ctx, J->up_bytes, J->down_bytes);
      if (rc) return rc;
      pinned = ctx->h_up;
    }
    std::memcpy(pinned, J->image, up);
  }
  return hip_check(ctx, hipMemcpyAsync(J->base, pinned, up, hipMemcpyHostToDevice, st), "upload");
}

int job_upload(rsl_ctx* ctx, Job* J, hipStream_t st, uint8_t* pinned) {
  int rc = job_upload_copy(ctx, J, st, pinned);
  if (!rc) rc = job_upload_digits(ctx, J, st);
  return rc;
}

int job_upload_digits(rsl_ctx* ctx, Job* J, hipStream_t st) {
  if (J->wdig_items.empty()) return RSL_OK;
  const int rc = ensure_tables(ctx, J->need_g, J->need_E, J->need_D);  // the prime constants; a no-op once grown
  if (rc) return rc;
  return hip_check(ctx, launch_wide_digits(reinterpret_cast<const DevProblem*>(J->base + J->probs_off),
                                           reinterpret_cast<const WorkItem*>(J->base + J->wdig_off),
                                           static_cast<int>(J->wdig_items.size()), J->wdig_lds, tables_of(ctx), st),
                   "wide digits");
}

int job_reset(rsl_ctx* ctx, Job* J, hipStream_t st) {
  if (J->status_bytes == 0) return RSL_OK;
  return hip_check(ctx, launch_copy_words(reinterpret_cast<uint32_t*>(J->base + J->status_off), nullptr,
                                          J->status_bytes / 4, st), "status reset");
}

int job_launch(rsl_ctx* ctx, Job* J, int mode, hipStream_t st, bool stage_events) {
  if (J->live.empty()) return RSL_OK;
  const DevTables T = tables_of(ctx);
  const DevProblem* probs = reinterpret_cast<const DevProblem*>(J->base + J->probs_off);
  auto items = [&](int s) { return reinterpret_cast<const WorkItem*>(J->base + J->items_off[s]); };
  auto wide = [&](int pass) { return reinterpret_cast<const WorkItem*>(J->base + J->wide_off[pass]); };
  int rc;
  if (mode == RSL_PLAIN) {
    for (size_t li = 0; li < J->live.size(); ++li) {
      const ProbLayout& L = J->lay[li];
      // the job-wide slot count: CRT kernels exist for 1-4, 6 and 8 slots, and
      // the CRT's LDS size was taken for that count
      const int ns = J->crt_ns;
      for (int s = 0; s < kNumStages; ++s) {
        const int cnt = L.item_end[s] - L.item_begin[s];
        const hipError_t e =
            s == kStageReduce && J->dev[li].evmf
                ? launch_reduce_tiles(J->dev[li].L_in <= 2 ? kReduceSlotsShort : kReduceSlotsLong, probs,
                                      items(s) + L.item_begin[s], cnt, T, st)
            : s == kStageEval ? launch_eval(eval_variant(J->dev[li]), probs, items(s) + L.item_begin[s], cnt,
                                          static_cast<size_t>(eval_stage_lds_words(J->dev[li])) * 4, T, st)
            : s == kStageConv || s == kStageStir
                ? launch_interp(s - kStageConv, probs, items(s) + L.item_begin[s], cnt, J->dev[li].D, T, st)
            : s == kStageCrt && J->crt_mm
                ? launch_crt_mm(probs, items(s) + L.item_begin[s], cnt, J->slot_np, T, st, true)
                : launch_stage(s, probs, items(s) + L.item_begin[s], cnt, J->stage_lds[s], ns, T, st, 1, true);
        if ((rc = hip_check(ctx, e, "launch"))) return rc;
      }
      for (int pass = 0; pass < 3; ++pass) {
        const int cnt = L.wide_end[pass] - L.wide_begin[pass];
        const int kp = (pass == 1 && J->wide_mfma) ? 3 : pass;
        if ((rc = hip_check(ctx, launch_crt_wide(kp, probs, wide(pass) + L.wide_begin[pass], cnt, J->wide_lds[pass], T, st,
                                                 true),
                            "launch")))
          return rc;
      }
    }
    return RSL_OK;
  }
  if (mode == RSL_BATCHED) {
    if (J->max_np > kMaxSlots)
      return fail(ctx, RSL_EINVAL, "the persistent schedule takes at most 256 primes per problem");
    if (J->any_schur)
      return fail(ctx, RSL_EINVAL, "the persistent schedule does not run the Schur evaluation");
    if (J->persist_lds > static_cast<size_t>(kLdsWords) * 4)
      return fail(ctx, RSL_EINVAL, "persistent launch needs more than 64 KB of LDS per workgroup");
    QueueDesc Q{};
    uint8_t* qb = J->base + J->queue_off;
    Q.state = reinterpret_cast<QueueState*>(qb);
    Q.tasks = reinterpret_cast<Task*>(qb + J->q_tasks);
    Q.ready = reinterpret_cast<int*>(qb + J->q_ready);
    Q.counters = reinterpret_cast<ProbCounters*>(qb + J->q_counters);
    Q.capacity = J->q_capacity;
    Q.crt_total = J->q_crt_total;
    Q.nprob = static_cast<int>(J->live.size());
    Q.wait_ticks = ctx->queue_wait_ticks;
    if (J->persist_grid == 0) {
      // at most two waiting waves per SIMD by default: idle waves only poll
      const int per_cu = std::min(8, persistent_blocks_per_cu(J->crt_ns, J->persist_lds));
      int cus = 256;
      hipDeviceProp_t prop;
      if (hipGetDeviceProperties(&prop, ctx->device) == hipSuccess) cus = prop.multiProcessorCount;
      J->persist_grid = std::max(1, per_cu * cus * std::max(1, J->tune.grid_mult));
    }
    if ((rc = hip_check(ctx, launch_copy_words(reinterpret_cast<uint32_t*>(qb),
                                               reinterpret_cast<const uint32_t*>(J->base + J->qinit_off),
                                               J->queue_bytes / 4, st),
                        "queue reset")))
      return rc;
    if (stage_events && (rc = hip_check(ctx, hipEventRecord(ctx->ev[0], st), "event"))) return rc;
    if ((rc = hip_check(ctx, launch_persistent(probs, Q, T, J->crt_ns, J->persist_grid, J->persist_lds, st),
                        "persistent launch")))
      return rc;
    if (stage_events)
      for (int s = 1; s <= kNumStages; ++s)
        if ((rc = hip_check(ctx, hipEventRecord(ctx->ev[s], st), "event"))) return rc;
    return RSL_OK;
  }
  for (int s = 0; s < kNumStages; ++s) {
    if (stage_events && (rc = hip_check(ctx, hipEventRecord(ctx->ev[s], st), "event"))) return rc;
    if (s == kStageReduce) {
      const int* rs = J->reduce_start;
      if ((rc = hip_check(ctx, launch_stage(s, probs, items(s), rs[1], J->stage_lds[s], J->crt_ns, T, st, 1, true),
                          "launch")) ||
          (rc = hip_check(ctx, launch_reduce_tiles(kReduceSlotsShort, probs, items(s) + rs[1], rs[2] - rs[1], T, st),
                          "launch")) ||
          (rc = hip_check(ctx, launch_reduce_tiles(kReduceSlotsLong, probs, items(s) + rs[2], rs[3] - rs[2], T, st),
                          "launch")))
        return rc;
      continue;
    }
    if (s == kStageEval) {
      const WorkItem* evs = reinterpret_cast<const WorkItem*>(J->base + J->evs_off);
      for (const Job::EvalRange& r : J->eval_ranges)
        if ((rc = hip_check(ctx, launch_eval(r.variant, probs, evs + r.begin, r.end - r.begin, r.lds, T, st),
                            "launch")))
          return rc;
      continue;
    }
    if (s == kStageConv || s == kStageStir) {
      if ((rc = hip_check(ctx, launch_interp(s - kStageConv, probs, items(s), static_cast<int>(J->items[s].size()),
                                             J->need_D, T, st),
                          "launch")))
        return rc;
      continue;
    }
    // column-sum CRT: several items per block once the launch still has a block
    // per CU or more
    const int crt_per = J->items[kStageCrt].size() >= 1024 ? kCrtItemsPerBlock : 1;
    const hipError_t e =
        s == kStageCrt && J->crt_mm
            ? launch_crt_mm(probs, items(s), static_cast<int>(J->items[s].size()), J->slot_np, T, st, true)
            : launch_stage(s, probs, items(s), static_cast<int>(J->items[s].size()), J->stage_lds[s], J->crt_ns, T, st,
                           crt_per, true);
    if ((rc = hip_check(ctx, e, "launch"))) return rc;
    if (s == kStageCrt)
      for (int pass = 0; pass < 3; ++pass)
        if ((rc = hip_check(ctx, launch_crt_wide((pass == 1 && J->wide_mfma) ? 3 : pass, probs, wide(pass),
                                                 static_cast<int>(J->wide_items[pass].size()),
                                                 J->wide_lds[pass], T, st, true), "launch")))
          return rc;
  }
  if (stage_events && (rc = hip_check(ctx, hipEventRecord(ctx->ev[kNumStages], st), "event"))) return rc;
  return RSL_OK;
}

int job_download(rsl_ctx* ctx, Job* J, uint8_t* host, hipStream_t st) {
  if (J->down_bytes == 0) return RSL_OK;
  return hip_check(ctx, hipMemcpyAsync(host, J->base + J->down_off, J->down_bytes, hipMemcpyDeviceToHost, st),
                   "download");
}

int job_decode(rsl_ctx* ctx, const Job& J, const uint8_t* host, rsl_result* out, int* status, rsl_counters* cnt) {
  std::vector<int> li_of(J.n, -1);
  for (size_t li = 0; li < J.live.size(); ++li) li_of[J.live[li]] = static_cast<int>(li);
  // statuses and degrees first; then the coefficients in blocks of about 64 KiB
  // over host threads, each read once (limbs needed and copy); then counters and
  // the first error in problem order
  std::vector<int> rcs(J.n, RSL_OK);
  struct Rows { int k, lo, hi, need; };
  std::vector<Rows> rows;
  std::vector<int> deg(J.n, -1);
  constexpr int kRowWords = 1 << 14;
  double words = 0.0;
  auto limbs_of = [&](int k) {
    return reinterpret_cast<const uint32_t*>(host + (J.lay[li_of[k]].out - J.down_off));
  };
  for (int k = 0; k < J.n; ++k) {
    const Plan& P = J.plans[k];
    rcs[k] = J.pstatus[k];
    if (rcs[k] || P.zero) {
      if (!rcs[k]) rcs[k] = decode_result(P, nullptr, &out[k]);
      continue;
    }
    const int* st = reinterpret_cast<const int*>(host + (J.lay[li_of[k]].status - J.down_off));
    if (st[0] & kErrQueueStall) { rcs[k] = RSL_EDEVICE; continue; }
    if (st[0] & kErrTooFewGoodPoints) { rcs[k] = RSL_EPRIMES; continue; }
    deg[k] = result_degree(limbs_of(k), P.D, P.L_out);
    const int step = std::max(1, kRowWords / P.L_out);
    for (int lo = 0; lo <= deg[k]; lo += step) rows.push_back({k, lo, std::min(deg[k] + 1, lo + step), 1});
    if (deg[k] < 0) rows.push_back({k, 0, 0, 1});
    words += (deg[k] + 1.0) * P.L_out;
  }
  parallel_for(static_cast<int>(rows.size()),
               std::max(1, static_cast<int>(rows.size() * static_cast<double>(kRowWords) / std::max(words, 1.0))),
               [&](int i) {
                 Rows& r = rows[i];
                 const int L = J.plans[r.k].L_out;
                 r.need = take_rows(limbs_of(r.k), L, r.lo, r.hi, &out[r.k], result_roomy(&out[r.k], L, deg[r.k]));
               });
  for (size_t i = 0; i < rows.size();) {
    const int k = rows[i].k, L = J.plans[k].L_out;
    int need = 1;
    for (; i < rows.size() && rows[i].k == k; ++i) need = std::max(need, rows[i].need);
    rcs[k] = finish_result(limbs_of(k), L, deg[k], need, result_roomy(&out[k], L, deg[k]), &out[k]);
  }
  int first = RSL_OK;
  for (int k = 0; k < J.n; ++k) {
    const int rc = rcs[k];
    const Plan& P = J.plans[k];
    if (!J.pstatus[k]) {
      cnt->problems += 1;
      if (!P.zero) {
        const ProbLayout& L = J.lay[li_of[k]];
        const int* st = reinterpret_cast<const int*>(host + (L.status - J.down_off));
        if (rc == RSL_EDEVICE) ctx->err = "persistent launch: a wave gave up waiting on the task queue";
        else if (rc == RSL_EPRIMES) ctx->err = "fewer than D+1 good points for a prime";
        else if (rc == RSL_ERANGE) ctx->err = "result buffer too small";
        cnt->pairs += static_cast<int64_t>(P.np) * (P.E + 1);
        cnt->bad_pairs += st[P.np + 1];
        cnt->bad_primes += P.bad_primes;
        for (int i = 0; i < P.np; ++i) cnt->slow_primes += st[1 + i];
      }
    }
    if (status) status[k] = rc;
    if (rc && !first) first = rc;
  }
  return first;
}

}  // namespace rsl
