"""The work a user of this library has it do, as cases that can be timed and compared.

Every case goes through the package's public entry points with host limbs in
and host limbs out (the library works on host data by its nature), except the
resident job, whose inputs stay on the device by the caller's choice:

  batch   PreparedBatch.run: n independent resultants in one call
  job     Job.run + rsl_job_results: a planned batch resident on the device
  serve   Server: a burst of requests, each waited for
  sqfree  Context.sqfree_part: the step after the resultant

Sizes are those of the repository's workloads and tests: total degrees 6..48,
8..64-bit coefficients, the curve-analysis discriminant, the large-coefficient
sets (2^128 .. 2^2048), and small ragged batches.  A case's shapes follow from
its own values; the seed draws the coefficients only.
"""

import ctypes
import math

import numpy as np

import paper_1010_1386_amd as rsl

_CTX = {}


def _context(name="main"):
    # one context for the program's life, as a program keeps it (its constant
    # tables are built by the first calls); a server owns a context of its own
    if name not in _CTX:
        _CTX[name] = rsl.Context(device=0, workspace_bytes=6 << 30, table_bytes=1 << 30)
    return _CTX[name]


def listed():
    return [
        # one small system, the solver's interactive call: latency and launches
        {"name": "one_d8", "kind": "batch", "n": 1, "dmin": 8, "dmax": 8, "bmin": 10, "bmax": 10, "sparse": 0.0,
         "var": "y", "mix": 1},
        # both projections of one dense degree-24 system, as the solver asks for them
        {"name": "pair_d24_xy", "kind": "batch", "n": 2, "dmin": 24, "dmax": 24, "bmin": 32, "bmax": 32,
         "sparse": 0.0, "var": "xy", "mix": 2},
        # one pair of very unequal odd degrees
        {"name": "one_d43_d19", "kind": "uneven", "df": 43, "dg": 19, "bits": 24, "var": "x"},
        # curve analysis: the discriminant of F (y^2 - h), 42 in y, degree bound 2054
        {"name": "curve_d40", "kind": "curve", "d": 40, "bits": 16},
        # many tiny systems in one call, ragged degrees
        {"name": "batch_61_small", "kind": "batch", "n": 61, "dmin": 3, "dmax": 11, "bmin": 8, "bmax": 40,
         "sparse": 0.5, "var": "mix", "mix": 5},
        # the batch workload: 512 pairs, half dense, half with zeroed coefficients
        {"name": "batch_512", "kind": "batch", "n": 512, "dmin": 6, "dmax": 32, "bmin": 8, "bmax": 64,
         "sparse": 0.5, "var": "y", "mix": 4},
        # degrees of the serving stream, both variables, as one call
        {"name": "stream_64", "kind": "batch", "n": 64, "dmin": 8, "dmax": 48, "bmin": 8, "bmax": 48,
         "sparse": 0.0, "var": "mix", "mix": 6},
        # the same stream through the server: a burst of requests
        {"name": "serve_40", "kind": "serve", "n": 40, "dmin": 8, "dmax": 48, "bmin": 8, "bmax": 48,
         "sparse": 0.0, "var": "mix", "mix": 7},
        # large coefficients, primes still in per-lane slots of the CRT
        {"name": "large_d9_2e512", "kind": "large", "d": 9, "shift": 512, "curves": 5},
        # large coefficients, thousands of primes
        {"name": "large_d15_2e2048", "kind": "large", "d": 15, "shift": 2048, "curves": 5},
        # the batch workload resident on the device, products on the matrix cores
        {"name": "job_256", "kind": "job", "n": 256, "dmin": 6, "dmax": 32, "bmin": 8, "bmax": 64, "sparse": 0.5,
         "var": "y", "mix": 8, "interp_mm": True},
        # square-free part of a resultant-sized polynomial q s^2
        {"name": "sqfree_d360", "kind": "sqfree", "dq": 120, "ds": 120, "bits": 64},
    ]


def draw(rng):
    kind = rng.choice(["batch", "batch", "batch", "pair", "uneven", "curve", "large", "job", "serve", "sqfree"])
    mix = rng.randrange(1 << 30)
    if kind == "pair":
        d = int(round(math.exp(rng.uniform(math.log(6), math.log(40)))))
        b = rng.randint(8, 64)
        return {"kind": "batch", "n": 2, "dmin": d, "dmax": d, "bmin": b, "bmax": b, "sparse": 0.0, "var": "xy",
                "mix": mix}
    if kind == "uneven":
        return {"kind": "uneven", "df": rng.randint(7, 44), "dg": rng.randint(7, 44), "bits": rng.randint(8, 64),
                "var": rng.choice("xy")}
    if kind == "curve":
        return {"kind": "curve", "d": rng.randint(6, 40), "bits": rng.randint(8, 16)}
    if kind == "large":
        d = rng.randint(6, 15)
        return {"kind": "large", "d": d, "shift": int(2 ** rng.uniform(7, 11)), "curves": rng.randint(2, 5)}
    if kind == "sqfree":
        return {"kind": "sqfree", "dq": rng.randint(12, 120), "ds": rng.randint(8, 120), "bits": rng.randint(8, 64)}
    n = int(round(math.exp(rng.uniform(0.0, math.log(300)))))
    top = 32 if n > 48 else 48
    dmin = rng.randint(3, 12)
    c = {"kind": kind, "n": n, "dmin": dmin, "dmax": rng.randint(dmin, top), "bmin": 8, "bmax": rng.randint(9, 64),
         "sparse": rng.choice([0.0, 0.5, 1.0]), "var": rng.choice(["y", "x", "mix"]), "mix": mix}
    if kind == "serve":
        c["n"] = 2 + n % 39
    if kind == "job":
        c["interp_mm"] = rng.choice([False, True])
    return c


# ------------------------------------------------------------------ inputs


def _shapes(case):
    """[(df, dg, bits_f, bits_g, zeroed, var)] of the case's problems (no seed)."""
    kind = case["kind"]
    if kind == "uneven":
        return [(case["df"], case["dg"], case["bits"], case["bits"], False, case["var"])]
    rng = np.random.default_rng(case["mix"])
    out = []
    for k in range(case["n"]):
        df, dg = (int(v) for v in rng.integers(case["dmin"], case["dmax"], size=2, endpoint=True))
        bf, bg = (int(v) for v in rng.integers(case["bmin"], case["bmax"], size=2, endpoint=True))
        v = case["var"]
        if v == "mix":
            v = "xy"[int(rng.integers(0, 2))]
        elif v == "xy":
            v = "yx"[k & 1]
        if case["var"] == "xy" and k & 1:
            df, dg, bf, bg = out[-1][:4]
        out.append((df, dg, bf, bg, k >= case["n"] * (1.0 - case["sparse"]), v))
    return out


def _total(rng, d, bits, zeroed):
    """Dense total degree d, signed `bits`-bit; zeroed: each coefficient 0 with probability 0.3."""
    lo, hi = -(1 << (bits - 1)), (1 << (bits - 1)) - 1
    a = rng.integers(lo, hi, size=(d + 1, d + 1), endpoint=True, dtype=np.int64)
    j, i = np.indices(a.shape)
    a[i + j > d] = 0
    if zeroed:
        a[rng.random(a.shape) < 0.3] = 0
        a[0, d] = a[0, d] or 1
    a[d, 0] = a[d, 0] or 1  # the y-degree is d
    return a


def _norm_bits(F):
    return math.log2(max(1, sum(abs(int(v)) for row in F for v in row)))


def _problems(case, seed):
    rng = np.random.default_rng([seed, 1010])
    kind = case["kind"]
    if kind == "curve":
        d = case["d"]
        F = _total(rng, d, case["bits"], False)
        h = rng.integers(-128, 127, size=7, endpoint=True)
        h[6] = h[6] or 1
        f = np.zeros((d + 3, d + 7), dtype=np.int64)
        f[2:, :d + 1] += F  # F y^2
        for k in range(7):
            f[:d + 1, k:k + d + 1] -= F * h[k]
        g = f[1:] * np.arange(1, d + 3, dtype=np.int64)[:, None]
        return [(f, g, "y")]
    if kind == "large":
        curves = []
        for _ in range(case["curves"]):
            F = [[int(v) << case["shift"] for v in row] for row in _total(rng, case["d"], 8, False)]
            F[0][0] += 1
            curves.append(F)
        return [(curves[a], curves[b], "y") for a in range(len(curves)) for b in range(a + 1, len(curves))]
    out = []
    for k, (df, dg, bf, bg, zeroed, v) in enumerate(_shapes(case)):
        if case.get("var") == "xy" and k & 1:  # the same system, eliminated in x
            out.append((out[-1][0], out[-1][1], v))
        else:
            out.append((_total(rng, df, bf, zeroed), _total(rng, dg, bg, zeroed), v))
    return out


def _bounds(case):
    """[(degree bound, limbs)] that hold for every problem of the case, from its values alone."""
    def limbs(m, n, bits_f, bits_g, terms_f, terms_g):
        return int(n * (bits_f + math.log2(terms_f)) + m * (bits_g + math.log2(terms_g)) + 3) // 32 + 1

    kind = case["kind"]
    if kind == "curve":
        d = case["d"]
        t = (d + 1) * (d + 2) // 2
        my, ny = d + 2, d + 1
        D = min((d + 6) * (my + ny), ny * (d + 6) + my * (d + 5) - my * ny)
        bits = case["bits"] + 8
        return [(D, limbs(my, ny, bits, bits + math.log2(d + 2), 8 * t, 8 * t))]
    if kind == "large":
        d = case["d"]
        t = (d + 1) * (d + 2) // 2
        n = case["curves"] * (case["curves"] - 1) // 2
        return [(d * d, limbs(d, d, 8 + case["shift"], 8 + case["shift"], t, t))] * n
    return [(df * dg, limbs(df, dg, bf, bg, (df + 1) * (df + 2) // 2, (dg + 1) * (dg + 2) // 2))
            for df, dg, bf, bg, _, _ in _shapes(case)]


# ------------------------------------------------------------------ states


def _own_buffers(args, bounds):
    """Point the C-ABI result records of `args` (PreparedBatch or Job) at one flat buffer."""
    flat = np.zeros(sum((D + 1) * L for D, L in bounds), dtype=np.int32)
    at = 0
    for k, (D, L) in enumerate(bounds):
        r = args.ra[k]
        r.cap_deg, r.limbs = D, L
        r.coeff = ctypes.cast(flat.ctypes.data + 4 * at, ctypes.POINTER(ctypes.c_uint32))
        at += (D + 1) * L
    return flat


def _degrees(args, n):
    return np.array([args.ra[k].deg for k in range(n)], dtype=np.int32)


def _pack(values):
    """Python ints as rows of equally many 32-bit limbs (two's complement)."""
    n = max((v.bit_length() + 1 for v in values), default=1)
    nb = 4 * ((n + 31) // 32)
    raw = b"".join(v.to_bytes(nb, "little", signed=True) for v in values)
    return np.frombuffer(raw, dtype=np.int32).reshape(len(values), nb // 4)


def _mul(a, b):
    """Product of two univariate integer polynomials by Kronecker substitution."""
    k = max(v.bit_length() for v in a) + max(v.bit_length() for v in b) + len(a).bit_length() + 2

    def pack(p):
        return sum(v << (k * i) for i, v in enumerate(p))
    return _unpack(pack(a) * pack(b), k, len(a) + len(b) - 1)


def _unpack(x, k, n):
    out, half, mask = [], 1 << (k - 1), (1 << k) - 1
    for _ in range(n):
        c = x & mask
        if c >= half:
            c -= 1 << k
        out.append(c)
        x = (x - c) >> k
    return out


def _factors(case, seed):
    rng = np.random.default_rng([seed, 1386])
    b = case["bits"] - 1

    def poly(d):
        v = [int(w) for w in rng.integers(-(1 << b), (1 << b) - 1, size=d + 1, endpoint=True, dtype=np.int64)]
        v[d] = v[d] or 1
        v[0] = v[0] or 1
        return v
    return poly(case["dq"]), poly(case["ds"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sqfree":
        q, s = _factors(case, seed)
        return {"kind": kind, "ctx": _context(), "r": _mul(q, _mul(s, s))}
    probs = _problems(case, seed)
    polys = {id(p): rsl.Poly(p) for f, g, _ in probs for p in (f, g)}  # inputs as limbs, packed once
    packed = [(polys[id(f)], polys[id(g)], v) for f, g, v in probs]
    if kind == "serve":
        if "server" not in _CTX:
            _CTX["server"] = rsl.Server(_context("serve"), budget_bytes=512 << 20, max_slots=64)
        return {"kind": kind, "server": _CTX["server"], "probs": packed, "bounds": _bounds(case)}
    if kind == "job":
        ctx = _context()
        job = ctx.job(packed, interp_mm=case["interp_mm"])
        lib = ctypes.CDLL(rsl.library_path())
        flat = _own_buffers(job, _bounds(case))
        return {"kind": kind, "ctx": ctx, "job": job, "n": len(packed), "flat": flat,
                "results": lib.rsl_job_results, "status": (ctypes.c_int * len(packed))()}
    pb = rsl.PreparedBatch(packed)
    return {"kind": kind, "ctx": _context(), "pb": pb, "n": len(packed), "flat": _own_buffers(pb, _bounds(case))}


def run(state):
    kind = state["kind"]
    if kind == "sqfree":
        q, g = state["ctx"].sqfree_part(state["r"])
        return {"q": _pack(q), "g": _pack(g)}
    if kind == "serve":
        s = state["server"]
        tickets = [s.submit(f, g, v) for f, g, v in state["probs"]]
        got = [s.wait(t, raw=True).raw() for t in tickets]
        return {"deg": np.array([d for d, _, _ in got], dtype=np.int32),
                "limbs": np.frombuffer(b"".join(raw.ljust(4 * (D + 1) * L, b"\0")
                                                for (_, _, raw), (D, L) in zip(got, state["bounds"])), dtype=np.int32)}
    if kind == "job":
        job = state["job"]
        job.run("staged")
        rc = state["results"](ctypes.c_void_p(state["ctx"].h.value), ctypes.c_void_p(job.h.value), job.ra,
                              state["status"])
        if rc:
            raise RuntimeError("rsl_job_results: %d" % rc)
        return {"deg": _degrees(job, state["n"]), "limbs": state["flat"]}
    state["pb"].run(state["ctx"], "auto")
    return {"deg": _degrees(state["pb"], state["n"]), "limbs": state["flat"]}


# ------------------------------------------------------------------ work


def work(case):
    """Input and output limbs once; two operations per modular multiply-add of the
    modular route at 30 bits a prime: evaluation, remainder sequences, interpolation
    and the CRT's limb products."""
    if case["kind"] == "sqfree":
        d = case["dq"] + 2 * case["ds"]
        bits = 3 * case["bits"] + 2 * math.log2(d)
        np_ = (bits + d + case["bits"] + case["ds"]) / 30
        return {"bytes": (d + 1) * bits / 8 + (case["dq"] + case["ds"] + 2) * (bits + case["bits"]) / 8,
                "flops": 2 * np_ * (2 * d * d + 2 * d * bits / 32)}
    if case["kind"] in ("curve", "large"):
        d = case["d"] + (2 if case["kind"] == "curve" else 0)
        bits = case["bits"] + 8 if case["kind"] == "curve" else 8 + case["shift"]
        shapes = [(d, d, bits, bits)] * len(_bounds(case))
    else:
        shapes = [s[:4] for s in _shapes(case)]
    nb = fl = 0.0
    for (df, dg, bf, bg), (D, _) in zip(shapes, _bounds(case)):
        tf, tg = (df + 1) * (df + 2) / 2, (dg + 1) * (dg + 2) / 2
        bits = dg * (bf + math.log2(tf) / 2) + df * (bg + math.log2(tg) / 2)
        primes = max(1.0, bits / 30)
        nb += (tf * bf + tg * bg + (D + 1) * bits) / 8
        fl += 2 * primes * ((D + 1) * (tf + tg + df * dg) + (D + 1) ** 2 + (D + 1) * bits / 32
                            + tf * bf / 32 + tg * bg / 32)
    return {"bytes": nb, "flops": fl}


# ------------------------------------------------------------------ exact values


def _content(v):
    g = 0
    for c in v:
        g = math.gcd(g, c)
    return g


def exact(case, seed):
    """Whole numbers from Python integers where that takes seconds: small single
    problems by a fraction-free determinant of the Sylvester matrix at x = 2^k
    (large enough that the value's digits are the coefficients), square-free
    parts from the factors."""
    if case["kind"] == "sqfree":
        q, s = _factors(case, seed)
        c = _content(s) * (1 if s[-1] > 0 else -1)
        return {"q": _pack(_mul([c * v for v in q], s)), "g": _pack([v // c for v in s])}
    if case["kind"] not in ("batch", "uneven") or max(max(s[:2]) for s in _shapes(case)) > 9 or len(
            _shapes(case)) > 2:
        return None
    degs, rows = [], []
    for (f, g, v), (D, L) in zip(_problems(case, seed), _bounds(case)):
        f, g = ([[int(c) for c in row] for row in (p if v == "y" else p.T)] for p in (f, g))
        k = 32 * L + 2
        a, b = ([sum(c << (k * i) for i, c in enumerate(row)) for row in p] for p in (f, g))
        while a[-1] == 0:
            a.pop()
        while b[-1] == 0:
            b.pop()
        m, n = len(a) - 1, len(b) - 1
        S = [[0] * i + a[::-1] + [0] * (n - 1 - i) for i in range(n)]
        S += [[0] * i + b[::-1] + [0] * (m - 1 - i) for i in range(m)]
        sign, prev = 1, 1
        for t in range(m + n):
            piv = next((r for r in range(t, m + n) if S[r][t]), None)
            if piv is None:
                prev = 0
                break
            if piv != t:
                S[t], S[piv], sign = S[piv], S[t], -sign
            for r in range(t + 1, m + n):
                S[r] = [0] * (t + 1) + [(S[t][t] * S[r][c] - S[r][t] * S[t][c]) // prev for c in range(t + 1, m + n)]
            prev = S[t][t]
        R = _unpack(sign * prev, k, D + 1)
        while R and R[-1] == 0:
            R.pop()
        degs.append(len(R) - 1)
        words = b"".join(c.to_bytes(4 * L, "little", signed=True) for c in R)
        rows.append(np.frombuffer(words + bytes(4 * L * (D + 1) - len(words)), dtype=np.int32))
    return {"deg": np.array(degs, dtype=np.int32), "limbs": np.concatenate(rows)}
