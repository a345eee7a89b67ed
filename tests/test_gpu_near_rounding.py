"""Rounding of the list pass's pair kernel, pair by pair: one system of isolated
pairs (nothing else within r_c of either), so that each near force gives back the
pair's coefficient 1/r^3 - 2 sum_l omega_l/s_l^2 e^{-r^2/s_l^2}, compared with long
double arithmetic at the same coordinates (FP32C: the fixed-point ones).

Roundings of single operations have no common sign, so the mean error over many pairs
shows what the coefficients of the sum of Gaussians are off by.  Tolerance: one unit
roundoff (2^-53, 2^-24) of 1/r^3, the rounding of a single constant of the sum's
size; the mean of 8,000 errors of some two units scatters by 0.03 of one."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R

pytestmark = pytest.mark.gpu


def _isolated_pairs(orc, prec, row, rc):
    """Near forces on the first of each pair along the pair's axis over its length, U_N,
    the pairs' r^2 in long double, and the split."""
    side, n = 20, 16000
    rng = np.random.default_rng(int(10 * rc))
    a = 2.2 * rc
    L = side * a
    grid = np.stack(np.unravel_index(np.arange(side ** 3), (side,) * 3), axis=1)
    mid = (grid + 0.5) * a
    r = rc * np.cbrt(rng.uniform(0.25 ** 3, 1.0, size=(side ** 3, 1)))
    e = rng.standard_normal((side ** 3, 3))
    e /= np.linalg.norm(e, axis=1, keepdims=True)
    pos = np.stack([mid - 0.5 * r * e, mid + 0.5 * r * e], axis=1).reshape(n, 3)
    q = np.tile([1.0, -1.0], n // 2)
    sog = R.rbsog_sog_table1(row, rc)
    s = R.System(pos, q, np.array([L, L, L]), rc, 8, seed=3, precision=prec, sog=sog)
    s.sample_k(1)
    _, E = s.forces()
    Fn, _ = s.components()
    s.close()
    if prec == R.RBSOG_FP32C:
        x = np.floor(pos / L * 2.0 ** 32).astype(np.longdouble) * (np.longdouble(L) / 2.0 ** 32)
    else:
        t = pos / L
        x = ((t - np.floor(t)) * L).astype(np.longdouble)
    d = x[1::2] - x[::2]
    r2 = np.sum(d * d, axis=1)
    # F on the first of a pair = -q_i q_j g d = g d
    got = np.sum(Fn[::2].astype(np.longdouble) * d, axis=1) / r2
    return got, E[0], r2, orc.SOG(sog.b, sog.sigma, sog.w0, sog.M)


@pytest.mark.parametrize("prec,unit", [(R.RBSOG_FP64, 2.0 ** -53), (R.RBSOG_FP32C, 2.0 ** -24)])
@pytest.mark.parametrize("row", [1, 2])
@pytest.mark.parametrize("rc", [2.0, 2.5, 3.5, 7.7, 9.0, 10.0])
def test_sum_of_gaussians_has_no_offset(orc, prec, unit, row, rc):
    got, _, r2, split = _isolated_pairs(orc, prec, row, rc)
    want = r2 ** np.longdouble(-1.5)
    for w, t in zip(split.omega, split.s):
        b = 1 / (np.longdouble(t) * np.longdouble(t))
        want = want - 2 * np.longdouble(w) * b * np.exp(-r2 * b)
    err = ((got - want) * r2 ** np.longdouble(1.5) / unit).astype(np.float64)
    print(f"row {row} rc {rc} prec {prec}: mean {err.mean():+.2f} rms {np.sqrt(np.mean(err ** 2)):.2f} units", flush=True)
    assert abs(err.mean()) < 1.0


@pytest.mark.parametrize("row", [1, 2])
@pytest.mark.parametrize("rc", [2.0, 2.5, 3.5, 7.7, 9.0, 10.0])
def test_energies_have_no_offset(orc, row, rc):
    """FP32C, U_N = -sum of the pairs' potentials: half a unit roundoff of the sum of
    1/r, what rounding one constant of the sum's size may take from every pair.  (FP64
    says nothing here: omega_l and s_l, which the library and the oracle each round to
    FP64 in their own formulas, move that sum by up to a unit of 2^-53 themselves.)"""
    _, U, r2, split = _isolated_pairs(orc, R.RBSOG_FP32C, row, rc)
    h = r2 ** np.longdouble(-0.5)
    for w, t in zip(split.omega, split.s):
        h = h - np.longdouble(w) * np.exp(-r2 / (np.longdouble(t) * np.longdouble(t)))
    err = float((np.longdouble(U) + h.sum()) / (r2 ** np.longdouble(-0.5)).sum() / 2.0 ** -24)
    print(f"row {row} rc {rc}: {err:+.2f} units", flush=True)
    assert abs(err) < 0.5
