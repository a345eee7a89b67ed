"""The FP32C structure factor keeps all 32 bits of a coordinate: positions on the
fixed-point grid itself, so that the expected phases m.u mod 2^32 are known to the
bit, and charges that pair.  Neighbours' coordinates differ by odd and by even
numbers of units, whose halves are not and are on the grid.

Tolerance: each phase is rounded to the 2^-23 turns of the hardware sine, by less
than 2 pi 2^-24 or, where a pair's half difference may leave out a bit (wave vectors
with |m_x| + |m_y| + |m_z| up to 256 only), than 2 pi 2^-23 of a radian.  Sums of n
such terms err by less than that part of their size."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R

from test_gpu_structure_factor import device_sf, rho_err

pytestmark = pytest.mark.gpu

TOL = 2.0 * np.pi * 2.0 ** -23


@pytest.mark.parametrize("n", [63, 2000, 20001])
@pytest.mark.parametrize("top", [30, 85, 86, 200, 2000, 20000, 2 * 10 ** 6, 2 ** 31 - 1])
def test_phases_use_every_bit_of_the_coordinates(n, top):
    rng = np.random.default_rng(n + top)
    u = rng.integers(0, 2 ** 32, size=(n, 3), dtype=np.uint64)
    u[n // 2:] = (u[:n - n // 2] + rng.integers(0, 4, size=(n - n // 2, 3), dtype=np.uint64)) % 2 ** 32
    q = np.where(rng.random(n) < 0.5, 1.0, -1.0)
    m = rng.integers(-top, top + 1, size=(130, 3))
    box = np.array([64.0, 32.0, 128.0])
    re, im = device_sf(u.astype(np.float64) / 2.0 ** 32 * box, q, box, m.astype(np.int32), R.RBSOG_FP32C)
    phase = np.zeros((len(m), n), dtype=np.uint64)
    for d in range(3):
        phase += m[:, d].astype(np.uint64)[:, None] * u[:, d][None, :]  # modulo 2^64
    t = (phase % 2 ** 32).astype(np.float64) * (2.0 * np.pi / 2.0 ** 32)
    err = rho_err(re, im, np.cos(t) @ q, np.sin(t) @ q)
    print(f"n {n} |m| <= {top}: {err:.2e}", flush=True)
    assert err < TOL
