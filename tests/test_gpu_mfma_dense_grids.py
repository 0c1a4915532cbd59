"""Matrix-core sums on grids whose knots are as many as the workgroups or more:
the split of the samples (shares of samples and of a gap per interval) against
the oracle and the vector path, alone and in a batch, down to single samples,
empty intervals and shares without samples.

Bars: the paths' own (binary64 1e-10, mixed 1e-5, of the largest |h|); the inner
product is the sum over the same samples; a batch gives the same bits.
"""
import numpy as np
import pytest

import oracle
from paper_2104_04582_amd import synth

pytestmark = pytest.mark.gpu
BAR = {"fp64": 1e-10, "mixed": 1e-5}


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2104_04582_amd import native
    native.load()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return native, torch, torch.device("cuda:0")


def draw(seed, l_max, n_max, n, K, k_max=None, grid="log", t0=0.0):
    rng = np.random.default_rng(seed)
    T = 10.0 * max(n, 4)
    if k_max is None:
        w = synth.draw_waveform(rng, synth.mode_list(2, l_max, n_max), T, K, 10.0)
    else:
        w = synth.draw_kerr(rng, synth.mode_list_kerr(2, l_max, k_max, n_max), T, K, 10.0)
    t = w.t_knots
    if grid == "ends":          # nearly all knots in the first and last thousandth
        s = np.linspace(-1.0, 1.0, K)
        t = T * 0.5 * (1.0 + np.sign(s) * (1.0 - 1e-3 * (1.0 - np.abs(s))))
        t[0], t[-1] = 0.0, T
    elif grid == "random":
        t = np.concatenate([[0.0], np.sort(rng.uniform(0.0, T, K - 2)), [T]])
    w.t_knots = t
    w.amp = synth._amp_at_knots(w.amp_poly, t, T)
    w.phi_phi = synth.chirp_phase(t, w.f0, w.tc)
    w.phi_r = w.kappa * w.phi_phi
    if k_max is not None:
        w.phi_theta = 0.93 * w.phi_phi
    w.t_start = t0 * T
    w.n_samples = min(n, synth.n_samples_for(T, w.dt, w.t_start))
    return w


LONG = [("fp64", dict(seed=1, l_max=7, n_max=31, n=262_144, K=1000)),
        ("fp64", dict(seed=2, l_max=10, n_max=30, n=262_145, K=600, grid="ends")),
        ("fp64", dict(seed=3, l_max=10, n_max=30, n=400_000, K=257, grid="random", t0=0.2)),
        ("mixed", dict(seed=4, l_max=3, n_max=31, n=262_144, K=1000)),
        ("mixed", dict(seed=5, l_max=6, n_max=16, n=300_007, K=700, grid="ends")),
        ("mixed", dict(seed=6, l_max=5, n_max=15, n=900_001, K=513, grid="random", t0=0.1)),
        ("mixed", dict(seed=7, l_max=8, n_max=12, n=262_144, K=5)),
        # operand tables (480 terms and more), whatever the length
        ("mixed", dict(seed=8, l_max=10, n_max=30, n=8_640, K=40)),
        ("mixed", dict(seed=9, l_max=7, n_max=31, n=129, K=300, grid="random")),
        ("mixed", dict(seed=10, l_max=6, n_max=31, n=300_000, K=1000, grid="ends", t0=0.1)),
        ("mixed", dict(seed=11, l_max=8, n_max=20, n=1, K=4)),
        ("mixed", dict(seed=12, l_max=9, n_max=25, n=100_000, K=150))]
KERR = [(p, dict(seed=20 + i, l_max=5, n_max=15, n=n, K=K, k_max=1, grid=grid))
        for p in ("fp64", "mixed")
        for i, (n, K, grid) in enumerate(((1, 5, "log"), (127, 40, "log"), (128, 300, "random"),
                                          (129, 4, "log"), (5_000, 900, "ends"), (8_640, 150, "log"),
                                          (40_000, 257, "random"), (60_000, 20, "ends")))]


def spline(plan, torch, dev, w):
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    if w.phi_theta is not None:
        return plan.spline_fit_kerr(w.t_knots, d(w.phi_phi), d(w.phi_theta), d(w.phi_r), w.lmn, d(w.amp))
    return plan.spline_fit(w.t_knots, d(w.phi_phi), d(w.phi_r), w.lmn, d(w.amp))


@pytest.mark.parametrize("prec,case", LONG + KERR,
                         ids=[f"{p} {c['n']} samples {c['K']} knots {c.get('grid', 'log')}" for p, c in LONG + KERR])
def test_dense_grids(env, prec, case):
    native, torch, dev = env
    w = draw(**case)
    rng = np.random.default_rng(9)
    out, ip = [], None
    for vec in (False, True):
        with native.Plan(0, prec, vector_only=vec) as plan:
            sp = spline(plan, torch, dev, w)
            o = torch.full((w.n_samples,), float("nan"), dtype=plan.out_dtype, device=dev)
            plan.mode_sum(sp, w.theta, w.phi, w.dt, w.n_samples, t_start=w.t_start, out=o)
            if not vec:
                data = torch.view_as_complex(torch.from_numpy(rng.standard_normal((w.n_samples, 2))).to(dev))
                ip = plan.inner_product(sp, w.theta, w.phi, w.dt, w.n_samples, data.to(plan.out_dtype),
                                        t_start=w.t_start).cpu().numpy()
                data = data.to(plan.out_dtype).cpu().numpy().astype(np.complex128)
            out.append(o.cpu().numpy().astype(np.complex128))
    got, vec = out
    assert np.all(np.isfinite(got))
    assert w.n_samples < 64 or not np.array_equal(got, vec)
    assert oracle.max_rel_error(got, vec) <= BAR[prec]
    st = native.host_interval_starts(w.t_knots, w.t_start, w.dt, w.n_samples)
    idx = set(rng.choice(w.n_samples, min(100, w.n_samples), replace=False).tolist())
    idx.update(int(s) + q for s in rng.choice(st[:-1], 60) for q in (-1, 0, 63, 64))
    idx = np.array(sorted(i for i in idx if 0 <= i < w.n_samples), dtype=np.int64)
    assert oracle.max_rel_error(got[idx], oracle.mode_sum_waveform(w, idx=idx)) <= BAR[prec]
    want = 2 * w.dt * np.array([np.sum((data.conj() * got).real), np.sum(np.abs(got) ** 2)])
    size = 2 * w.dt * np.array([np.sum(np.abs(data) * np.abs(got)), np.sum(np.abs(got) ** 2)])
    assert np.all(np.abs(ip - want) <= 1e-12 * size)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batch_on_dense_grids(env, prec):
    native, torch, dev = env
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ws = [draw(**c) for p, c in LONG if p == prec]
    ws.insert(1, draw(30, 3, 3, 700, 300, grid="random"))
    with native.Plan(0, prec) as plan:
        reqs, solo = [], []
        for w in ws:
            out = torch.empty(w.n_samples, dtype=plan.out_dtype, device=dev)
            reqs.append(dict(t_knots=w.t_knots, phi_phi=d(w.phi_phi), phi_r=d(w.phi_r), lmn=w.lmn,
                             amp=d(w.amp), theta=w.theta, phi=w.phi, dt=w.dt, n_samples=w.n_samples,
                             out=out, t_start=w.t_start))
            solo.append(plan.mode_sum(spline(plan, torch, dev, w), w.theta, w.phi, w.dt, w.n_samples,
                                      t_start=w.t_start))
        plan.batch(reqs)
        torch.cuda.synchronize()
        for q, s in zip(reqs, solo):
            assert torch.equal(torch.view_as_real(q["out"]), torch.view_as_real(s))


# lists whose operands cost more on so many knots than the products save
VECTOR = [("fp64", dict(seed=40, l_max=3, n_max=15, n=262_144, K=1000)),
          ("fp64", dict(seed=41, l_max=5, n_max=15, n=300_000, K=1000)),
          ("fp64", dict(seed=42, l_max=5, n_max=15, n=300_000, K=400, k_max=2)),
          ("mixed", dict(seed=43, l_max=5, n_max=3, n=1_000_000, K=1000)),
          ("mixed", dict(seed=44, l_max=5, n_max=8, n=1_000, K=900, k_max=2))]


@pytest.mark.parametrize("prec,case", VECTOR, ids=[f"{p} {c['n']} samples {c['K']} knots" for p, c in VECTOR])
def test_short_lists_on_dense_grids_stay_on_the_vector_kernel(env, prec, case):
    native, torch, dev = env
    w = draw(**case)
    out = []
    for vec in (False, True):
        with native.Plan(0, prec, vector_only=vec) as plan:
            out.append(plan.mode_sum(spline(plan, torch, dev, w), w.theta, w.phi, w.dt, w.n_samples).cpu().numpy())
    assert np.array_equal(out[0], out[1])
