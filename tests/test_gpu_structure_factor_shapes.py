"""The context-free structure factor where its launch shape changes: one chunk
or several, one wave's staging full or ragged, whole and partial k tiles, the
group limit of 1024 wave vectors, a stage's 1024 particles, charges that pair
and charges that do not, and wave vectors of any size.

Tolerances: FP64 sums of n unit phases err by about 1e-15 sqrt(n) of their
size, FP32C by the 2^-23-turn truncation of each phase (4e-7 of a radian RMS
per particle against sums of about sqrt(n)): 1e-11 and 1e-5 leave both room."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R

from test_gpu_structure_factor import device_sf, rho_err

pytestmark = pytest.mark.gpu

TOL = {R.RBSOG_FP64: 1e-11, R.RBSOG_FP32C: 1e-5}


@pytest.mark.parametrize("prec", [R.RBSOG_FP64, R.RBSOG_FP32C])
@pytest.mark.parametrize("n,nk", [(3, 1), (63, 64), (64, 65), (65, 63), (256, 128), (257, 128), (512, 64), (513, 64),
                                  (1024, 64), (1025, 64), (1023, 1024), (1025, 1025), (5000, 2111), (32768, 17),
                                  (70001, 1024), (600_000, 130)])
def test_shapes_match_oracle(orc, prec, n, nk):
    rng = np.random.default_rng(7 * n + nk)
    box = np.array([25.0, 21.0, 30.0])
    pos = rng.uniform(-0.5, 1.5, size=(n, 3)) * box
    q = rng.choice([1.0, -1.0, 2.0], size=n) if n % 2 else np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    m = rng.integers(-30, 31, size=(nk, 3)).astype(np.int32)
    re, im = device_sf(pos, q, box, m, prec)
    re_o, im_o = orc.structure_factor(pos, q, box, m)
    err = rho_err(re, im, re_o, im_o)
    print(f"n={n} nk={nk} prec={prec}: {err:.2e}", flush=True)
    assert err < TOL[prec]


@pytest.mark.parametrize("prec", [R.RBSOG_FP64, R.RBSOG_FP32C])
def test_wave_vectors_of_any_size(prec):
    """Positions on a grid of 1/1024 of the box: the phases of 32-bit wave
    vectors are exact, so the sums are known whatever the vectors' size."""
    rng = np.random.default_rng(3)
    n, nk = 3000, 200
    j = rng.integers(0, 1024, size=(n, 3))
    q = np.where(np.arange(n) < n // 2, 1.0, -1.0)
    m = rng.integers(-2 ** 31 + 1, 2 ** 31, size=(nk, 3))
    box = np.array([64.0, 32.0, 128.0])
    re, im = device_sf(j / 1024.0 * box, q, box, m.astype(np.int32), prec)
    t = 2.0 * np.pi * ((m @ j.T) % 1024) / 1024.0
    assert rho_err(re, im, np.cos(t) @ q, np.sin(t) @ q) < TOL[prec]
