"""GPU mode selector where a radix level leaves few candidates: they are ranked
among themselves (at most 64) or by another level (more).  The masks must be
those of the oracle."""
import numpy as np
import pytest

from oracle.mode_select import mode_select

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cluster", [2, 3, 63, 64, 65, 200])
@pytest.mark.parametrize("equal", [0, 1, 40])
def test_cut_inside_a_cluster(cluster, equal):
    """`cluster` powers that share their leading bits (relative spread 2^-12)
    straddle the threshold; `equal` of them are the same."""
    import torch
    from paper_2104_04582_amd import native
    rng = np.random.default_rng(100 * cluster + equal)
    K, M = 5, 1500
    amp = np.zeros((K, M, 2))
    eps = []
    for k in range(K):
        power = np.exp(rng.uniform(-20.0, 0.0, M))
        at = rng.choice(M, cluster, replace=False)
        power[at] = 0.01 * (1.0 + 2.0 ** -12 * rng.random(cluster))
        power[at[:equal]] = power[at[0]]
        ang = rng.uniform(0.0, 2 * np.pi, M)
        amp[k, :, 0], amp[k, :, 1] = np.sqrt(power) * np.cos(ang), np.sqrt(power) * np.sin(ang)
        above = power[power > 0.0101].sum() + power[at].sum() * rng.uniform(0.05, 0.95)
        eps.append(1.0 - above / power.sum())
    with native.Plan(0, "fp64") as plan:
        a = torch.from_numpy(amp).to("cuda:0")
        for k, e in enumerate(eps):
            got = plan.mode_select(a[k:k + 1].contiguous(), e).cpu().numpy()
            np.testing.assert_array_equal(got, mode_select(amp[k:k + 1], e))
            got = plan.mode_select(a, e).cpu().numpy()
            np.testing.assert_array_equal(got, mode_select(amp, e))
