"""The far force where its kernel shares a group's records among waves (16, 8,
4, 2 or none, by the number of groups and records), at the ends of the shares:
record counts that leave waves without records or with one to three records
beside groups of four, more than one stage of 256 records a wave, particle
counts off the groups of 64, several systems.  Against the oracle's far force
with the tolerances the far force has elsewhere: 1e-11 (FP64) and 1e-5 (FP32C)
relative RMS."""
import math

import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [(R.RBSOG_FP64, 1e-11), (R.RBSOG_FP32C, 1e-5)])
@pytest.mark.parametrize("sizes,P", [
    ([64], 2), ([130], 3), ([1000], 31), ([1002], 65), ([1000], 67), ([1000], 4357),  # 16 waves a group and fewer
    ([20002], 129), ([40000], 97), ([66000], 33), ([132000], 21), ([264000], 9),   # 8, 4, 2 and 1
    ([500, 64, 3070], 40)])
def test_far_split_matches_oracle(orc, prec, tol, sizes, P):
    rng = np.random.default_rng(P)
    pos, q, box, seeds = [], [], [], []
    for s, n in enumerate(sizes):
        L = max(10.0, (n / 0.1) ** (1 / 3))
        box.append(np.array([L, 1.25 * L, 0.9 * L]))
        pos.append(rng.random((n, 3)) * box[-1])
        q.append(np.where(np.arange(n) % 2 == 0, 1.0, -1.0))
        seeds.append(7 + s)
    sog = R.rbsog_sog_table1(2, 3.0)
    b = R.Batch(pos, q, box, 3.0, P, seeds, precision=prec)
    b.sample_k(1)
    b.forces()
    _, Ff = b.components()
    p0 = 0
    for s, n in enumerate(sizes):
        m = R.rbsog_get_kbatch(b.ctx, P, s)
        at = np.arange(n) if n <= 4000 else np.unique(np.concatenate([np.arange(70), np.arange(n - 70, n),
                                                                      rng.integers(0, n, 1000)]))
        Fo, _, _, _ = orc.far_rb(pos[s], q[s], box[s], orc.SOG(sog.b, sog.sigma, sog.w0, sog.M), m, P, targets=at)
        err = math.sqrt(float(np.sum((Ff[p0 + at] - Fo) ** 2) / np.sum(Fo ** 2)))
        print(f"n {n} P {P} prec {prec}: far relrms {err:.2e}", flush=True)
        assert err < tol
        p0 += n
    b.close()
