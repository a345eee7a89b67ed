"""Langevin steps whose far kernel opens the next step, against the same steps
one call at a time (each opened by the kick/drift kernel): the same values in
the same order, so positions, velocities and displacements are equal bit for
bit, whichever wave draws the noise."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R
from paper_2205_13824_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [R.RBSOG_FP64, R.RBSOG_FP32C])
@pytest.mark.parametrize("n,P", [(130, 30), (1002, 100), (20002, 70), (280000, 20)])
def test_fused_langevin_steps_equal_single_steps(prec, n, P):
    side = int(np.ceil(n ** (1 / 3)))
    L = (n / 0.1) ** (1 / 3)
    rng = np.random.default_rng(n)
    grid = np.stack(np.unravel_index(rng.permutation(side ** 3)[:n], (side,) * 3), axis=1)
    pos = (grid + 0.5 + rng.uniform(-0.25, 0.25, size=(n, 3))) * (L / side)
    q = np.where(np.arange(n) < n // 2, 1.0, -1.0)
    rng.shuffle(q)
    vel = W.maxwellian(n, 1.0, 5)
    out = []
    for calls in ([23], [1] * 23, [9, 1, 13]):
        s = R.System(pos, q, np.array([L, L, L]), 3.5, P, seed=4, precision=prec, device_chains=8)
        R.rbsog_set_thermostat(s.ctx, 2.0, 1.5, seed=11)
        R.rbsog_set_velocities(s.ctx, vel)
        R.rbsog_set_msd_origin(s.ctx)
        for k in calls:
            s.step(k, 2e-3)
        out.append((*R.rbsog_get_state(s.ctx, n), R.rbsog_get_msd(s.ctx)))
        s.close()
    print(f"n {n} prec {prec}: msd {out[0][2]}", flush=True)
    for o in out[1:]:
        for a, b in zip(out[0], o):
            np.testing.assert_array_equal(a, b)
