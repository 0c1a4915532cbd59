"""GPU parity of the matrix-core summation from the fold table: short and
middle mode lists and generic Kerr (one polar index after the other, joined by
a Horner recurrence in e^{-i Phi_theta}), at every compiled shape.

The operands are those of the matrix-core path (fp16 hi + lo, binary32 sums),
and the recurrence adds one binary32 rounding per polar index: the path's bars
hold, mismatch <= 1e-6 and max relative error <= 1e-5, against the oracle at
sampled outputs and against the vector path at every sample.
"""
import numpy as np
import pytest

import oracle
from paper_2104_04582_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2104_04582_amd import native
    native.load()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return native, torch, torch.device("cuda:0")


def draw(seed, l_max, n_max, n, K=9, k_max=None, keep=None, rough=False, offset=0.0):
    rng = np.random.default_rng(seed)
    T = max(10.0 * n, 3 * synth.DAY_S)
    if k_max is None:
        w = synth.draw_waveform(rng, synth.mode_list(2, l_max, n_max), T, K, 10.0)
    else:
        w = synth.draw_kerr(rng, synth.mode_list_kerr(2, l_max, k_max, n_max), T, K, 10.0)
    if keep is not None:
        sel = np.array([keep(*q) for q in w.lmn.tolist()])
        w.lmn, w.amp = w.lmn[sel].copy(), w.amp[:, sel].copy()
    if rough:
        w.amp = rng.standard_normal(w.amp.shape)
    w.t_start = offset * w.t_knots[1]
    w.n_samples = min(n, synth.n_samples_for(w.T, w.dt, w.t_start))
    return w


# shapes: row tiles of 8 signed m, steps of 16 |n|
CASES = [
    ("1x1", lambda: draw(1, 3, 9, 300_011)),
    ("2x1 rough", lambda: draw(3, 5, 8, 262_144, K=12, rough=True)),
    ("2x1 16 rows |n| 15", lambda: draw(4, 8, 15, 270_099, keep=lambda l, m, n: m % 2 == 0 and l <= 7)),
    ("2x2 |n| 16", lambda: draw(5, 4, 16, 440_001, offset=0.37)),
    ("2x2 |n| 31 short intervals", lambda: draw(6, 3, 31, 262_200, K=1000)),
    ("3x1", lambda: draw(7, 8, 9, 300_021, K=20)),
    ("3x2 gaps in m and n", lambda: draw(8, 10, 21, 280_000, rough=True,
                                         keep=lambda l, m, n: m in (0, 4, 7, 10) and n % 9 < 8 and l > 8)),
    ("kerr one sample", lambda: draw(2, 3, 15, 1, k_max=1)),
    ("kerr 1x1", lambda: draw(9, 3, 10, 30_000, k_max=1)),
    ("kerr 2x1 many samples", lambda: draw(10, 5, 6, 900_000, k_max=2)),
    ("kerr 2x2 odd k", lambda: draw(11, 7, 31, 8_001, k_max=3,
                                    keep=lambda l, m, k, n: k % 2 == 1)),
    ("kerr 3x2 rough", lambda: draw(12, 9, 30, 5_000, k_max=2, rough=True)),
    ("kerr 3x2 k > 0", lambda: draw(15, 10, 30, 300_003, K=30, offset=0.5, k_max=2,
                                    keep=lambda l, m, k, n: k > 0)),
    ("kerr k = 0", lambda: draw(14, 4, 9, 290_000, k_max=0)),
    # too few terms per polar index at this length, too few samples: vector kernel
    ("vector: 262143 samples", lambda: draw(16, 4, 16, 262_143)),
    ("vector: kerr k > 0", lambda: draw(13, 10, 30, 200_003, K=30, offset=0.5, k_max=2,
                                        keep=lambda l, m, k, n: k > 0)),
]


def spline(plan, torch, dev, w):
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    if w.phi_theta is not None:
        return plan.spline_fit_kerr(w.t_knots, d(w.phi_phi), d(w.phi_theta), d(w.phi_r), w.lmn, d(w.amp))
    return plan.spline_fit(w.t_knots, d(w.phi_phi), d(w.phi_r), w.lmn, d(w.amp))


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_terms_against_oracle_and_vector_path(env, case):
    native, torch, dev = env
    w = case[1]()
    out, ip = {}, {}
    rng = np.random.default_rng(7)
    data = torch.from_numpy(rng.standard_normal((w.n_samples, 2)).astype(np.float32)).to(dev)
    data = torch.view_as_complex(data)
    for vec in (False, True):
        with native.Plan(0, "mixed", vector_only=vec) as plan:
            sp = spline(plan, torch, dev, w)
            out[vec] = plan.mode_sum(sp, w.theta, w.phi, w.dt, w.n_samples, t_start=w.t_start)
            ip[vec] = plan.inner_product(sp, w.theta, w.phi, w.dt, w.n_samples, data,
                                         t_start=w.t_start)
            torch.cuda.synchronize()
    got, vec = (out[v].cpu().numpy().astype(np.complex128) for v in (False, True))
    idx = set(rng.choice(w.n_samples, min(300, w.n_samples), replace=False).tolist())
    for s in native.host_interval_starts(w.t_knots, w.t_start, w.dt, w.n_samples)[:-1]:
        idx.update(int(s) + d for d in (-1, 0, 1, 63, 64))
    idx = np.array(sorted(i for i in idx if 0 <= i < w.n_samples), dtype=np.int64)
    ref = oracle.mode_sum_waveform(w, idx=idx)
    for name, a, b in (("oracle", got[idx], ref), ("vector path", got, vec)):
        err, mm = oracle.max_rel_error(a, b), oracle.mismatch(a, b)
        print(f"    {case[0]} against {name}: max_rel_err={err:.3e} mismatch={mm:.3e}", flush=True)
        assert np.all(np.isfinite(a)) and mm <= 1e-6 and err <= 1e-5
    # two summation paths round differently: equal bits mean one path
    assert w.n_samples < 64 or np.array_equal(got, vec) == case[0].startswith("vector")
    # inner products are the sums over the same binary32 samples
    h, d = got, data.cpu().numpy().astype(np.complex128)
    want = np.array([2 * w.dt * np.sum((d.conj() * h).real), 2 * w.dt * np.sum(np.abs(h) ** 2)])
    size = 2 * w.dt * np.array([np.sum(np.abs(d) * np.abs(h)), np.sum(np.abs(h) ** 2)])
    assert np.all(np.abs(ip[False].cpu().numpy() - want) <= 1e-12 * size)


def test_batch_of_all_shapes_equals_single_sums(env):
    """One batch over every summation launch (vector, each matrix-core shape,
    operand tables): the same bits as each request by itself."""
    native, torch, dev = env
    ws = [c[1]() for c in CASES if "kerr" not in c[0]]
    ws += [draw(20, 2, 3, 9_000), draw(21, 10, 30, 12_345), draw(22, 3, 6, 6_000)]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    with native.Plan(0, "mixed") as plan:
        reqs, solo = [], []
        for w in ws:
            pp, pr, amp = d(w.phi_phi), d(w.phi_r), d(w.amp)
            out = torch.empty(w.n_samples, dtype=torch.complex64, device=dev)
            reqs.append(dict(t_knots=w.t_knots, phi_phi=pp, phi_r=pr, lmn=w.lmn, amp=amp,
                             theta=w.theta, phi=w.phi, dt=w.dt, n_samples=w.n_samples, out=out,
                             t_start=w.t_start))
            sp = plan.spline_fit(w.t_knots, pp, pr, w.lmn, amp)
            solo.append(plan.mode_sum(sp, w.theta, w.phi, w.dt, w.n_samples, t_start=w.t_start))
        plan.batch(reqs)
        torch.cuda.synchronize()
        for q, s in zip(reqs, solo):
            assert torch.equal(torch.view_as_real(q["out"]), torch.view_as_real(s))
