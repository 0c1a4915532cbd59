"""Performance cases of libfew: the calls a user's program makes, through the
binding's public entry points, over the range of sizes it makes them at.

  listed()   the named cases
  draw(rng)  one more case of the same ranges
  prepare    what a program holds before the call: inputs on the GPU, the plan,
             the output buffers (and the fitted spline where it is kept)
  run        one pass
  work       bytes and flops that a pass cannot do without
  exact      the same outputs in binary64 by plain numpy and torch

A case is a plain dict.  Common keys: op, precision, modes, knots, days, dt.
Mode lists: all (l, m, n) with l <= l_max, |n| <= n_max (and |k| <= k_max for
generic Kerr); `top` > 0 keeps that many modes of largest power, as the mode
selector leaves them.  Sizes follow bench.py and synth.py: one day to four
years, 20 to 150 knots, 5 to 15 s cadence.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2104_04582_amd import native, synth

DEV = "cuda:0"
YEAR_DAYS = 365.25


def _case(name, op, precision, l_max, n_max, knots, days, dt, **more):
    c = {"name": name, "op": op, "precision": precision, "l_max": l_max, "n_max": n_max,
         "k_max": 0, "top": 0, "knots": knots, "days": days, "dt": dt, "requests": 1, "eps": 1e-5}
    c.update(more)
    return c


def listed():
    return [
        # the smallest waveform in use (one day, 132 modes): host path, launches, latency
        _case("day 132 modes mixed", "step", "mixed", 4, 5, 40, 1.0, 10.0),
        # a small generic-Kerr waveform in binary64 (660 modes, one day)
        _case("day kerr 660 modes fp64", "kerr", "fp64", 4, 5, 40, 1.0, 10.0, k_max=2),
        # the headline waveform: the full Schwarzschild set over one year
        _case("year 3843 modes mixed", "step", "mixed", 10, 30, 100, YEAR_DAYS, 10.0),
        # the same in binary64, the accuracy reference a user checks against
        _case("year 3843 modes fp64", "step", "fp64", 10, 30, 100, YEAR_DAYS, 10.0),
        # the longest request: four years, written in the barycentre frame
        _case("4 years ssb mixed", "ssb", "mixed", 10, 30, 100, 4 * YEAR_DAYS, 10.0),
        # after mode selection: a few hundred modes, ragged length, 15 s cadence
        _case("0.6 year top 230 mixed", "step", "mixed", 10, 30, 77, 219.3, 15.0, top=230),
        # selected modes in binary64 on a dense grid of knots
        _case("0.3 year top 611 fp64", "step", "fp64", 10, 30, 137, 113.7, 10.0, top=611),
        # generic Kerr: nine times the mode count, one year
        _case("year kerr 34587 modes mixed", "kerr", "mixed", 10, 30, 100, YEAR_DAYS, 10.0, k_max=4),
        # likelihood evaluations over extrinsic parameters: spline kept, <d|h> and <h|h>
        _case("year inner mixed", "inner", "mixed", 10, 30, 100, YEAR_DAYS, 10.0),
        # a posterior's worth of uneven waveforms in one call
        _case("batch of 24 mixed", "batch", "mixed", 10, 30, 150, 2 * YEAR_DAYS, 10.0, requests=24),
        # concurrent requests through the server, submitted together
        _case("served 6 fp64", "served", "fp64", 10, 30, 90, 0.2 * YEAR_DAYS, 15.0, requests=6),
        # choosing the modes of a waveform (the step before the sum)
        _case("select 3843 modes", "select", "fp64", 10, 30, 100, YEAR_DAYS, 10.0),
    ]


def _log_uniform(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def _samples(c):
    return synth.n_samples_for(c["days"] * synth.DAY_S, c["dt"])


def draw(rng):
    """A case of the listed ranges.  The waveform is shortened until it costs
    no more than the one-year generic-Kerr sum (binary64 counted twice)."""
    op = rng.choice(["step", "step", "step", "ssb", "kerr", "inner", "batch", "served", "select"])
    precision = rng.choice(["mixed", "mixed", "fp64"])
    l_max, n_max = rng.randint(3, 10), rng.randint(3, 30)
    k_max = rng.randint(1, 4) if op == "kerr" else 0
    days = _log_uniform(rng, 0.7, 4 * YEAR_DAYS)
    c = {"op": op, "precision": precision, "l_max": l_max, "n_max": n_max, "k_max": k_max,
         "top": 0, "knots": rng.randint(20, 150), "days": days,
         "dt": rng.choice([5.0, 10.0, 10.0, 15.0]), "requests": 1, "eps": 1e-5}
    if op == "select":
        # lists long enough that some modes fall below the threshold
        c["l_max"], c["n_max"] = rng.randint(6, 10), rng.randint(12, 30)
        c["eps"] = _log_uniform(rng, 1e-5, 1e-2)
    if op in ("batch", "served"):
        c["requests"] = rng.randint(2, 24 if op == "batch" else 8)
        c["days"] = min(c["days"], (2.0 if op == "batch" else 0.5) * YEAR_DAYS)
    if rng.random() < 0.5 and op != "kerr":
        c["top"] = min(int(_log_uniform(rng, 10, 3843)), len(synth.mode_list(2, l_max, n_max)))
    cap = 3.2e6 * 11529
    cost = lambda: c["requests"] * _samples(c) * (_terms(_modes(c)) + 100) * (
        2 if precision == "fp64" else 1)
    while op != "select" and (cost() > cap or c["requests"] * _samples(c) > 3e7):
        c["days"] *= 0.8
    return c


# ---- inputs ------------------------------------------------------------------
def _modes(c):
    if c["op"] == "kerr":
        return synth.mode_list_kerr(2, c["l_max"], c["k_max"], c["n_max"])
    return synth.mode_list(2, c["l_max"], c["n_max"])


def _waveform(c, rng):
    T = c["days"] * synth.DAY_S
    if c["op"] == "kerr":
        return synth.draw_kerr(rng, _modes(c), T, c["knots"], c["dt"])
    w = synth.draw_waveform(rng, _modes(c), T, c["knots"], c["dt"])
    return synth.top_modes(w, c["top"]) if c["top"] else w


def _waveforms(c, seed):
    """The waveforms of a case: one, or the uneven requests of a batch (lengths,
    knots and mode counts spread as in synth.uneven_instance).  Their sizes
    belong to the case, their values to the seed."""
    if c["op"] not in ("batch", "served"):
        return [_waveform(c, np.random.default_rng([seed, 1]))]
    out = []
    for i in range(c["requests"]):
        size = np.random.default_rng([c["requests"], c["knots"], i])
        d = dict(c, days=c["days"] * size.uniform(0.125, 1.0),
                 knots=int(size.integers(max(4, c["knots"] // 3), c["knots"] + 1)))
        n_all = len(_modes(c))
        d["top"] = min(n_all, c["top"] or int(round(math.exp(size.uniform(math.log(10), math.log(n_all))))))
        out.append(_waveform(d, np.random.default_rng([seed, 2, i])))
    return out


def _sky(seed):
    """(theta_S, phi_S, theta_K, phi_K) of the detector-frame calls."""
    r = np.random.default_rng([seed, 3])
    return (math.acos(r.uniform(-1, 1)), r.uniform(0, 2 * math.pi),
            math.acos(r.uniform(-1, 1)), r.uniform(0, 2 * math.pi))


def _data(n, seed, dtype):
    """Strain-like data of the inner products: white noise."""
    g = torch.Generator(device=DEV).manual_seed(int(seed) + 17)
    return torch.complex(torch.randn(n, generator=g, device=DEV, dtype=torch.float64),
                         torch.randn(n, generator=g, device=DEV, dtype=torch.float64)).to(dtype)


class State:
    """A program's plan, inputs and buffers; the plan goes with the state."""

    def __del__(self):
        try:
            torch.cuda.synchronize()
            self.plan.close()
        except Exception:
            pass


def prepare(case, seed):
    s = State()
    ws = _waveforms(case, seed)
    s.op, s.eps = case["op"], case["eps"]
    s.plan = native.Plan(0, case["precision"], hbm_budget_bytes=2 << 30)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    s.reqs = []
    for w in ws:
        s.reqs.append(dict(t_knots=w.t_knots, phi_phi=dev(w.phi_phi), phi_r=dev(w.phi_r), lmn=w.lmn,
                           amp=dev(w.amp), theta=w.theta, phi=w.phi, dt=w.dt, n_samples=w.n_samples))
        if s.op not in ("inner", "select"):
            s.reqs[-1]["out"] = torch.empty(w.n_samples, dtype=s.plan.out_dtype, device=DEV)
    q = s.reqs[0]
    if s.op == "kerr":
        s.phi_theta = dev(ws[0].phi_theta)
    elif s.op == "ssb":
        s.sky = _sky(seed)
    elif s.op == "inner":
        s.data = _data(q["n_samples"], seed, s.plan.out_dtype)
        s.dh_hh = torch.empty(2, dtype=torch.float64, device=DEV)
        s.spline = s.plan.spline_fit(q["t_knots"], q["phi_phi"], q["phi_r"], q["lmn"], q["amp"])
    elif s.op == "select":
        s.keep = torch.empty(len(q["lmn"]), dtype=torch.int32, device=DEV)
    return s


def run(s):
    plan, q = s.plan, s.reqs[0]
    if s.op == "batch":
        plan.batch(s.reqs)
        return [r["out"] for r in s.reqs]
    if s.op == "served":
        for t in [plan.submit(**r) for r in s.reqs]:
            plan.wait(t)
        return [r["out"] for r in s.reqs]
    if s.op == "select":
        return plan.mode_select(q["amp"], s.eps, keep=s.keep)
    if s.op == "inner":
        plan.inner_product(s.spline, q["theta"], q["phi"], q["dt"], q["n_samples"], s.data,
                           out2=s.dh_hh)
        # in the precision of the waveform they were formed from
        return s.dh_hh if plan.precision == "fp64" else s.dh_hh.to(torch.float32)
    if s.op == "kerr":
        sp = plan.spline_fit_kerr(q["t_knots"], q["phi_phi"], s.phi_theta, q["phi_r"], q["lmn"],
                                  q["amp"])
    else:
        sp = plan.spline_fit(q["t_knots"], q["phi_phi"], q["phi_r"], q["lmn"], q["amp"])
    if s.op == "ssb":
        plan.mode_sum_ssb(sp, *s.sky, q["dt"], q["n_samples"], out=q["out"])
    else:
        plan.mode_sum(sp, q["theta"], q["phi"], q["dt"], q["n_samples"], out=q["out"])
    sp.free()
    return q["out"]


# ---- work ----------------------------------------------------------------------
def _terms(modes):
    """Distinct signed (m, [k,] n) of a mode list and its mirrors."""
    a = np.asarray(modes, dtype=np.int64)[:, 1:]
    return len(np.unique(np.concatenate([a, -a[a[:, 0] > 0]]), axis=0))


def work(case):
    """Inputs once, outputs once; per folded term and sample the complex cubic
    in a real variable (12 flop) and one complex multiply-add (8)."""
    size = 16 if case["precision"] == "fp64" else 8
    b = f = 0.0
    for w in _waveforms(case, 1):
        amp = 16.0 * w.K * w.M
        if case["op"] == "select":
            b, f = amp + 4.0 * w.M, 3.0 * w.K * w.M
            break
        b += size * w.n_samples + (0.0 if case["op"] == "inner" else amp)
        f += 20.0 * _terms(w.lmn) * w.n_samples
    return {"bytes": b, "flops": f}


# ---- binary64 reference ------------------------------------------------------------
def _swsh(l, m, theta, phi):
    """-2Y_lm by the explicit sum over powers of cos, sin of theta / 2 (extended
    precision; the sum alternates)."""
    f = math.factorial
    c, s = np.cos(np.longdouble(theta) / 2), np.sin(np.longdouble(theta) / 2)
    v = np.longdouble(0)
    for r in range(max(0, m - 2), min(l + m, l - 2) + 1):
        k = f(l + m) * f(l - m) * f(l + 2) * f(l - 2) // 1
        den = f(l + m - r) * f(r) * f(r - m + 2) * f(l - 2 - r)
        v += (-1) ** r * np.sqrt(np.longdouble(k)) / np.longdouble(den) * \
            c ** (2 * l + m - 2 - 2 * r) * s ** (2 * r - m + 2)
    v *= np.sqrt(np.longdouble(2 * l + 1) / (4 * np.longdouble(math.pi)))
    return complex(float(v)) * complex(math.cos(m * phi), math.sin(m * phi))


def _cubics(t, y):
    """Not-a-knot cubics of the columns of y [K, S]: [4, K-1, S] in x = t - t_i."""
    K, h = len(t), np.diff(t)
    d = np.diff(y, axis=0) / h[:, None]
    A, b = np.zeros((K, K)), np.zeros_like(y)
    A[0, 0], A[0, 1] = h[1], h[0] + h[1]
    b[0] = ((h[0] + 2 * (h[0] + h[1])) * h[1] * d[0] + h[0] ** 2 * d[1]) / (h[0] + h[1])
    for r in range(1, K - 1):
        A[r, r - 1], A[r, r], A[r, r + 1] = h[r], 2 * (h[r - 1] + h[r]), h[r - 1]
        b[r] = 3 * (h[r] * d[r - 1] + h[r - 1] * d[r])
    A[-1, -1], A[-1, -2] = h[-2], h[-1] + h[-2]
    b[-1] = (h[-1] ** 2 * d[-2] + (2 * (h[-2] + h[-1]) + h[-1]) * h[-2] * d[-1]) / (h[-2] + h[-1])
    s = np.linalg.solve(A, b)
    hh = h[:, None]
    return np.stack([y[:-1], s[:-1], (3 * d - 2 * s[:-1] - s[1:]) / hh,
                     (s[:-1] + s[1:] - 2 * d) / hh ** 2])


def _reference(w, theta, phi, factor=1.0):
    """h of one waveform, complex128 on the GPU: the folded sum over signed
    (m, k, n), interval by interval, phases relative to the interval's knot."""
    lm = np.asarray(w.lmn, dtype=np.int64)
    l, m, n = lm[:, 0], lm[:, 1], lm[:, -1]
    k = lm[:, 2] if lm.shape[1] == 4 else np.zeros_like(l)
    Y = {(a, b): _swsh(a, b, theta, phi) for a, b in set(zip(l.tolist(), m.tolist()))
         | set(zip(l.tolist(), (-m).tolist()))}
    co = _cubics(w.t_knots, w.amp.reshape(w.K, -1))
    A = torch.from_numpy(co[..., 0::2] + 1j * co[..., 1::2]).to(DEV)          # [4, K-1, M]
    up = np.array([Y[a, b] for a, b in zip(l.tolist(), m.tolist())]) * factor
    dn = np.array([Y[a, -b] for a, b in zip(l.tolist(), m.tolist())]) * (-1.0) ** (l + k) * factor
    mirror = m > 0
    rows_m, rows_k, cols = (np.unique(np.concatenate([v, -v])) for v in (m, k, n))
    at = lambda a, b, c: ((np.searchsorted(rows_k, b) * len(rows_m) + np.searchsorted(rows_m, a))
                          * len(cols) + np.searchsorted(cols, c))
    C = torch.zeros(4, w.K - 1, len(rows_k) * len(rows_m) * len(cols), dtype=torch.complex128,
                    device=DEV)
    dev = lambda v: torch.from_numpy(v).to(DEV)
    C.index_add_(2, dev(at(m, k, n)), A * dev(up))
    if mirror.any():
        C.index_add_(2, dev(at(-m, -k, -n)[mirror]), A[:, :, dev(mirror)].conj() * dev(dn[mirror]))
    C = C.view(4, w.K - 1, len(rows_k), len(rows_m), len(cols))
    ph = [_cubics(w.t_knots, np.asarray(p)[:, None])[..., 0]
          for p in (w.phi_phi, w.phi_r, w.phi_theta) if p is not None]
    two_pi = 2 * np.longdouble("3.14159265358979323846264338327950288")
    knot = [np.remainder(np.asarray(p, dtype=np.longdouble), two_pi).astype(np.float64)
            for p in (w.phi_phi, w.phi_r, w.phi_theta) if p is not None]
    t = w.t_start + np.arange(w.n_samples, dtype=np.float64) * w.dt
    first = np.concatenate([[0], np.searchsorted(t, w.t_knots[1:-1]), [w.n_samples]])
    h = torch.empty(w.n_samples, dtype=torch.complex128, device=DEV)
    wave = lambda idx, g: torch.polar(torch.ones((), dtype=torch.float64, device=DEV).expand(
        len(idx), len(g)), -torch.outer(dev(idx.astype(np.float64)), g))
    for i in range(w.K - 1):
        for a in range(int(first[i]), int(first[i + 1]), 65536):
            b = min(a + 65536, int(first[i + 1]))
            x = dev(t[a:b] - w.t_knots[i])
            g = [torch.remainder(((p[3, i] * x + p[2, i]) * x + p[1, i]) * x, 2 * math.pi) + y[i]
                 for p, y in zip(ph, knot)]
            F, E = wave(cols, g[1]), wave(rows_m, g[0])
            T = wave(rows_k, g[2]) if len(g) == 3 else None
            tot = torch.zeros(b - a, dtype=torch.complex128, device=DEV)
            for q in range(len(rows_k)):
                S = torch.zeros(len(rows_m), b - a, dtype=torch.complex128, device=DEV)
                for p in (3, 2, 1, 0):
                    S = S * x + C[p, i, q] @ F
                S = (S * E).sum(0)
                tot += S if T is None else S * T[q]
            h[a:b] = tot
    return h


def exact(case, seed):
    ws = _waveforms(case, seed)
    w = ws[0]
    if case["op"] in ("batch", "served"):
        return [_reference(v, v.theta, v.phi) for v in ws]
    if case["op"] == "select":
        p = w.amp[:, :, 0] ** 2 + w.amp[:, :, 1] ** 2
        keep = np.zeros(w.M, dtype=np.int32)
        for row in p:
            order = np.argsort(-row, kind="stable")
            c = np.add.accumulate(row[order])
            keep[order[np.concatenate([[0.0], c[:-1]]) < (1.0 - case["eps"]) * c[-1]]] = 1
        return torch.from_numpy(keep)
    if case["op"] == "inner":
        h = _reference(w, w.theta, w.phi)
        d = _data(w.n_samples, seed, torch.complex64 if case["precision"] == "mixed"
                  else torch.complex128).to(torch.complex128)
        two_dt = 2.0 * w.dt
        return torch.stack([two_dt * torch.sum(d.real * h.real + d.imag * h.imag),
                            two_dt * torch.sum(h.real ** 2 + h.imag ** 2)])
    if case["op"] == "ssb":
        # viewing angles and polarisation factor of the detector frame
        ts, ps, tk, pk = _sky(seed)
        R = np.array([math.sin(ts) * math.cos(ps), math.sin(ts) * math.sin(ps), math.cos(ts)])
        S = np.array([math.sin(tk) * math.cos(pk), math.sin(tk) * math.sin(pk), math.cos(tk)])
        psi = math.atan2(math.cos(ts) * math.sin(tk) * math.cos(ps - pk) - math.sin(ts) * math.cos(tk),
                         math.sin(tk) * math.sin(ps - pk))
        return _reference(w, math.acos(max(-1.0, min(1.0, -float(R @ S)))), -math.pi / 2,
                          -complex(math.cos(2 * psi), -math.sin(2 * psi)))
    return _reference(w, w.theta, w.phi)
