"""GPU parity of the binary64 matrix-core summation: every compiled shape and
every way of forming the cubic (two, three or four powers in binary64
products, blocks of 32 or 16 samples, the rest in one or three fp16 products).

What is not summed in binary64 stays below 2^-52 of the largest coefficient,
and the powers of the harmonics are recurrences of at most 16 steps, 2^-49: far
below the phases' rounding (2^-53 pi times |m| + |n| + |k| <= 50, 2^-44).  The
binary64 path's bar holds, max relative error <= 1e-10 of the largest |h|,
against the oracle at sampled outputs and against the vector kernel at every sample.
"""
import numpy as np
import pytest

import oracle
from paper_2104_04582_amd import synth

pytestmark = pytest.mark.gpu
BAR = 1e-10


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2104_04582_amd import native
    native.load()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return native, torch, torch.device("cuda:0")


def draw(seed, l_max, n_max, n, K=9, k_max=None, rough=0.0, flat=None, offset=0.0, keep=None):
    rng = np.random.default_rng(seed)
    T = max(10.0 * n, synth.DAY_S)
    if k_max is None:
        w = synth.draw_waveform(rng, synth.mode_list(2, l_max, n_max), T, K, 10.0)
    else:
        w = synth.draw_kerr(rng, synth.mode_list_kerr(2, l_max, k_max, n_max), T, K, 10.0)
    if keep is not None:
        sel = np.array([bool(keep(*q)) for q in w.lmn.tolist()])
        w.lmn, w.amp = w.lmn[sel].copy(), w.amp[:, sel].copy()
    if rough:
        w.amp = w.amp * (1.0 + rough * rng.standard_normal(w.amp.shape))
    if flat is not None:
        w.amp = w.amp[:1] + flat * (w.amp - w.amp[:1])
    w.dt = T / n
    w.n_samples = n
    if offset:
        w.t_start = offset * w.t_knots[1]
        w.n_samples = synth.n_samples_for(w.T, w.dt, w.t_start)
    return w


def rough_end(w):
    """Smooth but for the last knot."""
    w.amp[-1] *= 1.5
    return w


CASES = [
    # amplitudes that vary by `flat` allow two powers, or longer blocks
    ("1x1 two powers", lambda: draw(2, 3, 15, 270_001, K=4, flat=1e-3)),
    ("2x1 two powers, blocks of 16", lambda: draw(3, 5, 15, 300_000, K=12, flat=0.5)),
    ("2x2 three powers", lambda: draw(4, 7, 26, 275_000, K=30, offset=0.4)),
    ("2x2 four powers", lambda: draw(5, 7, 31, 262_144, K=1000, rough=1.0)),
    ("3x1 gaps", lambda: draw(6, 10, 15, 300_000, K=6, keep=lambda l, m, n: m not in (2, 5) and n % 7)),
    ("3x2 short intervals", lambda: draw(7, 10, 30, 263_000, K=700, rough=1e-2)),
    # many samples, several rounds per wave
    ("3x2 many samples", lambda: draw(8, 10, 30, 800_017, K=100)),
    ("3x2 smooth and rough", lambda: rough_end(draw(9, 8, 30, 270_000, K=8, flat=1e-5))),
    ("kerr one sample", lambda: draw(1, 3, 9, 1, k_max=1)),
    ("kerr 2x1 very smooth", lambda: draw(10, 4, 5, 10_000, K=10, k_max=2, flat=1e-6)),
    ("kerr 3x2 k > 0", lambda: draw(11, 8, 30, 60_001, K=4, k_max=2, keep=lambda l, m, k, n: k > 0)),
    ("kerr 1x1 rough", lambda: draw(12, 3, 14, 5_000, K=20, k_max=1, rough=1.0, offset=0.3)),
    ("kerr k = 0", lambda: draw(13, 3, 15, 266_000, k_max=0)),
    # few of the cells filled, too few samples: vector kernel
    ("vector: 262143 samples", lambda: draw(15, 10, 30, 262_143)),
    ("vector: top terms", lambda: draw(14, 7, 20, 80_000, keep=lambda l, m, n: l == 7 and m < 3)),
]


def spline(plan, torch, dev, w):
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    if w.phi_theta is not None:
        return plan.spline_fit_kerr(w.t_knots, d(w.phi_phi), d(w.phi_theta), d(w.phi_r), w.lmn, d(w.amp))
    return plan.spline_fit(w.t_knots, d(w.phi_phi), d(w.phi_r), w.lmn, d(w.amp))


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_f64_against_oracle_and_vector_path(env, case):
    native, torch, dev = env
    w = case[1]()
    out, ip = {}, {}
    rng = np.random.default_rng(7)
    data = torch.view_as_complex(torch.from_numpy(rng.standard_normal((w.n_samples, 2))).to(dev))
    for vec in (False, True):
        with native.Plan(0, "fp64", vector_only=vec) as plan:
            sp = spline(plan, torch, dev, w)
            out[vec] = plan.mode_sum(sp, w.theta, w.phi, w.dt, w.n_samples, t_start=w.t_start)
            ip[vec] = plan.inner_product(sp, w.theta, w.phi, w.dt, w.n_samples, data,
                                         t_start=w.t_start)
            torch.cuda.synchronize()
    got, vec = (out[v].cpu().numpy() for v in (False, True))
    idx = set(rng.choice(w.n_samples, min(300, w.n_samples), replace=False).tolist())
    for s in native.host_interval_starts(w.t_knots, w.t_start, w.dt, w.n_samples)[:-1]:
        idx.update(int(s) + d for d in (-1, 0, 1, 63, 64))
    idx = np.array(sorted(i for i in idx if 0 <= i < w.n_samples), dtype=np.int64)
    ref = oracle.mode_sum_waveform(w, idx=idx)
    for name, a, b in (("oracle", got[idx], ref), ("vector path", got, vec)):
        err = oracle.max_rel_error(a, b)
        print(f"    {case[0]} against {name}: max_rel_err={err:.3e}", flush=True)
        assert np.all(np.isfinite(a)) and err <= BAR
    # two summation paths round differently: equal bits mean one path
    assert w.n_samples < 64 or np.array_equal(got, vec) == case[0].startswith("vector")
    h, d = got, data.cpu().numpy()
    want = np.array([2 * w.dt * np.sum((d.conj() * h).real), 2 * w.dt * np.sum(np.abs(h) ** 2)])
    size = 2 * w.dt * np.array([np.sum(np.abs(d) * np.abs(h)), np.sum(np.abs(h) ** 2)])
    assert np.all(np.abs(ip[False].cpu().numpy() - want) <= 1e-12 * size)


def test_batch_equals_single_sums(env):
    """One batch over the vector launch and every binary64 matrix launch: the
    same bits as each request by itself."""
    native, torch, dev = env
    ws = [c[1]() for c in CASES if "kerr" not in c[0]]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    with native.Plan(0, "fp64") as plan:
        reqs, solo = [], []
        for w in ws:
            pp, pr, amp = d(w.phi_phi), d(w.phi_r), d(w.amp)
            out = torch.empty(w.n_samples, dtype=torch.complex128, device=dev)
            reqs.append(dict(t_knots=w.t_knots, phi_phi=pp, phi_r=pr, lmn=w.lmn, amp=amp,
                             theta=w.theta, phi=w.phi, dt=w.dt, n_samples=w.n_samples, out=out,
                             t_start=w.t_start))
            sp = plan.spline_fit(w.t_knots, pp, pr, w.lmn, amp)
            solo.append(plan.mode_sum(sp, w.theta, w.phi, w.dt, w.n_samples, t_start=w.t_start))
        plan.batch(reqs)
        torch.cuda.synchronize()
        for q, s in zip(reqs, solo):
            assert torch.equal(torch.view_as_real(q["out"]), torch.view_as_real(s))
