"""The cell lists that a step and an evaluation build, at the sizes where the
build changes its kernels: batches that one block re-sorts inside a step (up to
8,192 particles and 3,072 cells) and larger ones, cells that a thread ranks
(up to 16 particles), a wave ranks in one pass (64) or in several, and counters
scanned by one block or by two kernels.  The expected order is exact: slots by
(cell, id) with cell = floor(u nc / 2^32) of the quantised coordinates."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R

pytestmark = pytest.mark.gpu


def _expected(x, box, start):
    nc = round((len(start) - 1) ** (1 / 3))
    assert nc ** 3 == len(start) - 1
    u = np.minimum(np.floor(x / box * 2.0 ** 32), 2.0 ** 32 - 1).astype(np.uint64)
    c = ((u * np.uint64(nc)) >> np.uint64(32)).astype(np.int64)
    cell = c[:, 0] + nc * (c[:, 1] + nc * c[:, 2])
    return np.lexsort((np.arange(len(x)), cell)), np.concatenate([[0], np.cumsum(np.bincount(cell, minlength=nc ** 3))])


@pytest.mark.parametrize("prec", [R.RBSOG_FP64, R.RBSOG_FP32C])
@pytest.mark.parametrize("n,density,rc", [
    (1000, 0.1, 3.5), (1030, 0.1, 3.5), (8192, 0.1, 3.5), (8194, 0.1, 3.5),    # ends of the one-block range
    (4096, 0.1, 5.0), (4096, 0.1, 8.0), (9000, 0.1, 11.0),                     # some 16, 60 and 160 in a cell
    (2700, 0.1, 1.9), (2700, 0.1, 1.8),                                        # about 3,072 cells
    (12000, 0.1, 1.95), (12000, 0.1, 1.9), (12000, 0.1, 0.85), (3000, 0.005, 1.0)])  # some 12,288, 131,072 and more
def test_build_order(prec, n, density, rc):
    rng = np.random.default_rng(n)
    L = (n / density) ** (1 / 3)
    side = int(np.ceil(n ** (1 / 3)))
    grid = np.stack(np.unravel_index(rng.permutation(side ** 3)[:n], (side,) * 3), axis=1)
    pos = (grid + 0.5 + rng.uniform(-0.25, 0.25, size=(n, 3))) * (L / side)
    q = np.where(np.arange(n) < n // 2, 1.0, -1.0)
    box = np.array([L, L, L])
    s = R.System(pos, q, box, rc, 10, seed=3, precision=prec, device_chains=4)
    s.forces()
    v = rng.standard_normal((n, 3))
    v *= 300.0 * rc / np.linalg.norm(v, axis=1, keepdims=True)  # 0.3 r_c a step: every step builds
    for steps in (0, 1, 9):  # a call's own evaluation, one step, a chunk of steps
        if steps:
            R.rbsog_set_velocities(s.ctx, v)
            s.step(steps, 1e-3)
        x, _ = R.rbsog_get_state(s.ctx, n)
        start, order = R.rbsog_debug_cells(s.ctx, n)
        want_order, want_start = _expected(x, box, start)
        print(f"n {n} rc {rc} prec {prec} steps {steps}: {len(start) - 1} cells, "
              f"largest {np.diff(start).max()}", flush=True)
        np.testing.assert_array_equal(start, want_start)
        np.testing.assert_array_equal(order, want_order)
    s.close()
