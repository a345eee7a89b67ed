"""Transfers between the caller's arrays and the state: the order is changed
on the device, small arrays pass through pinned memory (up to 512 KiB in all,
10,922 particles for two arrays and 21,845 for one), larger ones directly.
Everything here is exact: the same doubles in the caller's order."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R
from paper_2205_13824_amd import workloads as W

pytestmark = pytest.mark.gpu


def _system(n, prec):
    rng = np.random.default_rng(n)
    side = int(np.ceil(n ** (1 / 3)))
    grid = np.stack(np.unravel_index(np.arange(side ** 3), (side,) * 3), axis=1)[rng.permutation(side ** 3)[:n]]
    box = np.array([2.1544346900318843 * max(side, 4)] * 3)
    pos = (grid + 0.5 + rng.uniform(-0.2, 0.2, size=(n, 3))) * 2.1544346900318843
    q = np.where(np.arange(n) < n // 2, 1.0, -1.0)
    return pos, q, box, R.System(pos, q, box, 3.5, 16, seed=5, precision=prec)


@pytest.mark.parametrize("prec", [R.RBSOG_FP64, R.RBSOG_FP32C])
@pytest.mark.parametrize("n", [2, 64, 258, 10922, 10924, 21844, 21848, 30000])
def test_state_and_forces_keep_the_callers_order(n, prec):
    pos, q, box, s = _system(n, prec)
    s.sample_k(2)
    s.forces()  # the state is in cell order from here on
    rng = np.random.default_rng(n + 1)
    new = pos + rng.integers(-2, 3, size=(n, 3)) * box  # images of the same particles
    vel = W.maxwellian(n, 1.0, seed=n)
    R.rbsog_set_positions(s.ctx, new)
    R.rbsog_set_velocities(s.ctx, vel)
    x, v = R.rbsog_get_state(s.ctx, n)
    t = new / box
    assert np.array_equal(x, (t - np.floor(t)) * box)
    assert np.array_equal(v, vel)
    K, _ = R.rbsog_get_kinetic(s.ctx)
    assert abs(K[0] - 0.5 * np.sum(vel * vel)) <= 1e-12 * K[0]
    F, E = s.forces()
    Fn, Ff = s.components()
    assert np.array_equal(F, Fn + Ff)
    assert np.array_equal(E, R.rbsog_get_energy(s.ctx))
    ids = np.arange(n)[:: max(1, n // 50)]
    fn, ff = R.rbsog_get_forces_subset(s.ctx, ids)
    assert np.array_equal(fn, Fn[ids]) and np.array_equal(ff, Ff[ids])
    s.close()


@pytest.mark.parametrize("n", [64, 30000])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_a_refused_array_leaves_the_state(n, bad):
    pos, q, box, s = _system(n, R.RBSOG_FP64)
    s.sample_k(2)
    F0, _ = s.forces()
    x0, v0 = R.rbsog_get_state(s.ctx, n)
    for setter in (R.rbsog_set_positions, lambda c, a: R.rbsog_set_velocities(c, a)):
        arr = pos.copy()
        arr[n // 3, 1] = bad
        arr[n - 1, 2] = bad
        with pytest.raises(R.RbsogError) as e:
            setter(s.ctx, arr)
        assert e.value.status == -7 and f"particle {n // 3} " in str(e.value)
        x1, v1 = R.rbsog_get_state(s.ctx, n)
        assert np.array_equal(x0, x1) and np.array_equal(v0, v1)
        setter(s.ctx, pos if setter is R.rbsog_set_positions else np.zeros((n, 3)))  # and the next one is taken
    s.close()


def test_builds_are_counted_as_they_happen():
    pos, q, box, s = _system(3000, R.RBSOG_FP32C)
    s.sample_k(6)
    assert R.rbsog_info(s.ctx)["list_builds"] == 0
    s.forces()
    assert R.rbsog_info(s.ctx)["list_builds"] == 1
    state = R.rbsog_save_state(s.ctx)
    R.rbsog_set_positions(s.ctx, pos)
    s.step(2, 1e-4)
    assert R.rbsog_info(s.ctx)["list_builds"] == 2
    R.rbsog_load_state(s.ctx, state)
    assert R.rbsog_info(s.ctx)["list_builds"] == 1
    s.close()
