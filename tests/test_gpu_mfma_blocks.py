"""GPU parity of the matrix-core summation where it writes the cubic about the
centre of blocks of samples (smooth amplitudes over long intervals) and where
it keeps the interval's four coefficients (rough amplitudes, short intervals).

Blocks leave out at most 2^-25 of a row pair's largest coefficient per term and
round the block slope (at most 2^-11 of it) to fp16, 2^-23 together, which is
below the rounding of the harmonics: the matrix-core path's bars hold, mismatch
<= 1e-6 and max relative error <= 1e-5, against the oracle at sampled outputs
and against the vector path at every sample.
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


def smooth(seed, days, K, dt, offset=0.0, n_max=30):
    w = synth.draw_waveform(np.random.default_rng(seed), synth.mode_list(2, 10, n_max),
                            days * synth.DAY_S, K, dt)
    w.t_start = offset * w.t_knots[1]
    w.n_samples = synth.n_samples_for(w.T, dt, w.t_start)
    return w


def rough(seed, K, n):
    w = smooth(seed, 10.0, K, 10.0)
    w.amp = np.random.default_rng(seed + 1).standard_normal(w.amp.shape)
    w.dt = w.T / n
    w.n_samples = n
    return w


def one_rough_knot(seed):
    """Smooth but for one knot: blocks in most intervals, none around it."""
    w = smooth(seed, 200.0, 40, 30.0)
    w.amp[20] *= 1.5
    return w


CASES = [
    # blocks of many rounds, of a few, and too short to use (static tables)
    ("300 days 100 knots", lambda: smooth(60, 300.0, 100, 10.0)),
    ("40 days 12 knots", lambda: smooth(61, 40.0, 12, 10.0)),
    ("ragged 23 days 7 knots", lambda: smooth(62, 23.3, 7, 7.3, offset=0.61)),
    ("9 days 5 knots n 16..31", lambda: smooth(63, 9.0, 5, 5.0, n_max=31)),
    ("1 day 4 knots", lambda: smooth(64, 1.0, 4, 2.0)),
    # rough data: static tables, every power with all products
    ("rough 6 knots", lambda: rough(65, 6, 30_011)),
    ("rough 30 knots", lambda: rough(66, 30, 20_000)),
    ("one rough knot", lambda: one_rough_knot(67)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_blocks_and_static_tables_against_oracle(env, case):
    native, torch, dev = env
    w = case[1]()
    assert native.host_mfma_path(w.lmn)
    ins = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (w.phi_phi, w.phi_r, w.amp)]
    out = {}
    for vec in (False, True):
        with native.Plan(0, "mixed", vector_only=vec) as plan:
            sp = plan.spline_fit(w.t_knots, ins[0], ins[1], w.lmn, ins[2])
            out[vec] = plan.mode_sum(sp, w.theta, w.phi, w.dt, w.n_samples, t_start=w.t_start)
            torch.cuda.synchronize()
    got, vec = (out[v].cpu().numpy().astype(np.complex128) for v in (False, True))
    rng = np.random.default_rng(7)
    idx = set(rng.choice(w.n_samples, min(400, w.n_samples), replace=False).tolist())
    for s in native.host_interval_starts(w.t_knots, w.t_start, w.dt, w.n_samples)[:-1]:
        idx.update(int(s) + d for d in (-1, 0, 1, 63, 64, 127, 128))
    idx = np.array(sorted(i for i in idx if 0 <= i < w.n_samples), dtype=np.int64)
    ref = oracle.mode_sum_waveform(w, idx=idx)
    for name, a, b in (("oracle", got[idx], ref), ("vector path", got, vec)):
        err, mm = oracle.max_rel_error(a, b), oracle.mismatch(a, b)
        print(f"    {case[0]} against {name}: max_rel_err={err:.3e} mismatch={mm:.3e}", flush=True)
        assert np.all(np.isfinite(a)) and mm <= 1e-6 and err <= 1e-5
