"""Mixed lists that lie far from n = 0: the matrix-core sum forms e^{-i n Phi_r}
as a power of the sample's binary32 e^{-i Phi_r} (an error that grows with |n|),
the vector path walks each segment from its exact phase.  Whichever path a list
takes, its error is no larger than the vector path's: the rms over the samples
and six draws, with 1/8 for the spread of such a mean (six draws of an error
whose rms varies by less than 30 % from draw to draw).
"""
import numpy as np
import pytest

import oracle
from paper_2104_04582_amd import synth

pytestmark = pytest.mark.gpu

# (name, l_max, condition on (m, n), k_max, samples, matrix cores)
CASES = [
    ("n 20..31", 10, lambda m, n: 20 <= n, None, 600_000, False),
    ("|n| > 20", 7, lambda m, n: abs(n) > 20, None, 600_000, False),
    ("n 6..16", 10, lambda m, n: 6 <= n <= 16, None, 1_000_000, False),
    ("m >= 9, n 12..31", 11, lambda m, n: m >= 9 and n >= 12, None, 3_000_000, False),
    ("kerr n 18..30", 10, lambda m, n: 18 <= n < 31, 2, 400_000, False),
    # the vector path's walk is as long as the powers
    ("n 0..31", 10, lambda m, n: n >= 0, None, 600_000, True),
    ("n -5..25", 6, lambda m, n: -5 <= n <= 25, None, 600_000, True),
    ("|n| < 16", 5, lambda m, n: abs(n) < 16, None, 300_000, True),
    ("kerr |n| < 13", 6, lambda m, n: abs(n) < 13, 1, 20_000, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_no_less_accurate_than_the_vector_path(case):
    import torch
    from paper_2104_04582_amd import native
    name, l_max, keep, k_max, n, matrix = case
    dev = torch.device("cuda:0")
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    sq = np.zeros(2)
    for seed in range(6):
        rng = np.random.default_rng(seed)
        lm = synth.mode_list(2, l_max, 31) if k_max is None else synth.mode_list_kerr(2, l_max, k_max, 31)
        lm = lm[[bool(keep(q[1], q[-1])) for q in lm.tolist()]]
        w = (synth.draw_waveform if k_max is None else synth.draw_kerr)(rng, lm, 10.0 * n, 60, 10.0)
        w.amp = synth._amp_at_knots(rng.standard_normal(w.amp_poly.shape), w.t_knots, w.T)
        idx = np.sort(rng.choice(n, 300, replace=False))
        ref = oracle.mode_sum_waveform(w, idx=idx)
        out = []
        for vec in (False, True):
            with native.Plan(0, "mixed", vector_only=vec) as plan:
                if k_max is None:
                    sp = plan.spline_fit(w.t_knots, d(w.phi_phi), d(w.phi_r), w.lmn, d(w.amp))
                else:
                    sp = plan.spline_fit_kerr(w.t_knots, d(w.phi_phi), d(w.phi_theta), d(w.phi_r),
                                              w.lmn, d(w.amp))
                out.append(plan.mode_sum(sp, w.theta, w.phi, w.dt, n).cpu().numpy()[idx])
        size = np.max(np.abs(ref))
        sq += [np.mean(np.abs(o - ref) ** 2) / size ** 2 for o in out]
        assert np.array_equal(out[0], out[1]) != matrix
    rms = np.sqrt(sq / 6)
    print(f"    {name}: rms error {rms[0]:.2e}, vector path {rms[1]:.2e}", flush=True)
    assert rms[0] <= 1.125 * rms[1]
