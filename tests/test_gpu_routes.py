"""Which kernels an evaluation takes, by what rbsog_debug_routes reports, at the sizes
and options where the choice changes: the list pass's pair kernel by the split (the
results of its forms agree, so that only the report tells them apart) and the waves
that share a far group's records."""
import numpy as np
import pytest

from paper_2205_13824_amd import rbsog as R

pytestmark = pytest.mark.gpu

F64, F32C = R.RBSOG_FP64, R.RBSOG_FP32C


def _batch(sizes, P, prec, rc=3.0, rows=None, **kw):
    rng = np.random.default_rng(sum(sizes))
    pos, q, box = [], [], []
    for n in sizes:
        L = max(10.0, (n / 0.1) ** (1 / 3))
        box.append(np.array([L, L, L]))
        pos.append(rng.random((n, 3)) * L)
        q.append(np.where(np.arange(n) % 2 == 0, 1.0, -1.0))
    sogs = [R.rbsog_sog_table1(row, rc) for row in rows] if rows else None
    return R.Batch(pos, q, box, rc, P, list(range(len(sizes))), precision=prec, sogs=sogs, **kw)


def _routes(b, stepping=True):
    r = R.rbsog_debug_routes(b.ctx, stepping)
    b.close()
    return r


@pytest.mark.parametrize("prec", [F64, F32C])
@pytest.mark.parametrize("rc", [1.0, 3.5, 4.9])
@pytest.mark.parametrize("rows,form", [([1], 1), ([2], 1), ([3], 0), ([4], 0), ([5], 0), ([2, 1, 2], 1), ([2, 3, 1], 0)])
def test_pair_kernel_of_the_list_pass(prec, rc, rows, form):
    assert _routes(_batch([200] * len(rows), 8, prec, rc=rc, rows=rows))["near_form"] == form


def test_pair_kernel_of_the_core_shell_table():
    assert _routes(_batch([200], 8, F32C, near_table=True))["near_form"] == 2


# the waves that test_gpu_far_split.py's cases are about
@pytest.mark.parametrize("sizes,P,f64,f32", [([64], 2, 1, 1), ([1000], 31, 4, 4), ([1002], 65, 16, 16),
                                             ([1000], 4357, 16, 16), ([20002], 129, 16, 8), ([40000], 97, 8, 4),
                                             ([66000], 33, 4, 2), ([132000], 21, 2, 1), ([264000], 9, 1, 1),
                                             ([500, 64, 3070], 40, 8, 8),
                                             # systems of two groups each: 480, 512 and 1,026 of them
                                             ([66] * 240, 100, 16, 8), ([66] * 256, 100, 16, 8), ([66] * 513, 100, 4, 2)])
def test_waves_of_a_far_group(sizes, P, f64, f32):
    assert _routes(_batch(sizes, P, F64))["far_waves"] == f64
    assert _routes(_batch(sizes, P, F32C))["far_waves"] == f32


# two streams from 5e7 (FP64 2.2e7) particles x wave vectors on, up to 4e9; one block
# re-sorts steps of up to 8,192 particles
@pytest.mark.parametrize("prec,sizes,P,streams,one", [(F32C, [8192], 100, 1, 1), (F32C, [8194], 100, 1, 0),
                                                      (F32C, [100000], 500, 1, 0), (F32C, [100000], 502, 2, 0),
                                                      (F64, [100000], 220, 1, 0), (F64, [100000], 222, 2, 0),
                                                      (F64, [4000, 90], 100, 1, 1)])
def test_streams_and_shared_launches(prec, sizes, P, streams, one):
    b = _batch(sizes, P, prec)
    calls = R.rbsog_debug_routes(b.ctx, False)
    assert (calls["streams"], calls["shared"], calls["one_block"]) == (streams, 2 - streams, 0)
    steps = _routes(b)
    assert (steps["streams"], steps["shared"], steps["one_block"]) == (streams, 2 - streams, one)


def test_room_is_checked():
    b = _batch([100], 8, F32C)
    out = np.zeros(8, dtype=np.int32)
    for args in ((None, 1), (R._ptr(out), 0), (R._ptr(out), len(R.ROUTES) + 1)):
        assert R.lib().rbsog_debug_routes(b.ctx, 1, *args) == -1
    b.close()


# 480 chunks of particles beside the near part, 512 where the structure factor is alone
# (one stream, above 4e9 pairs too)
@pytest.mark.parametrize("prec,n,P,skin,chunks", [(F32C, 400000, 100, None, 512), (F32C, 400000, 200, None, 480),
                                                  (F64, 200000, 100, None, 512), (F64, 200000, 200, None, 480),
                                                  (F32C, 400000, 100, 0.0, 480), (F32C, 400000, 10100, None, 512)])
def test_chunks_of_the_structure_factor(prec, n, P, skin, chunks):
    b = _batch([n], P, prec, skin=skin)
    assert R.rbsog_info(b.ctx)["rho_chunk"] == -(-n // chunks)
    b.close()


# ragged systems of a batch stay within the 512 blocks that the device holds at once
# (their last chunks would make more of 512 of the mean size), equal ones that fit keep
# the 512
RAGGED = [500 + 2 * ((37 * i * i) % 3251) for i in range(40)]


@pytest.mark.parametrize("prec", [F64, F32C])
@pytest.mark.parametrize("sizes,chunks", [(RAGGED, 480), ([51200] * 4, 512), ([50200, 51000, 51800, 51800], 480)])
def test_chunks_of_a_batch(prec, sizes, chunks):
    b = _batch(sizes, 66, prec)
    chunk = R.rbsog_info(b.ctx)["rho_chunk"]
    assert chunk == -(-sum(sizes) // chunks)
    assert sum(-(-n // chunk) for n in sizes) <= 512
    b.close()


@pytest.mark.parametrize("sizes", [RAGGED])
def test_k_tiles_of_a_batch(sizes):
    b = _batch(sizes, 103, F64)
    assert R.rbsog_info(b.ctx)["rho_ktile"] == 2
    b.close()


# FP64 blocks of fewer k tiles where that lightens the fullest CU, not where every step
# builds: 391 chunks of 4 tiles make 782 blocks of 2 or 1,564 of 1
@pytest.mark.parametrize("prec,n,P,skin,ktile", [(F64, 100000, 200, None, 1), (F64, 100000, 200, 0.0, 4),
                                                 (F64, 1000, 100, None, 1), (F64, 1000, 100, 0.0, 1),
                                                 (F32C, 100000, 200, None, 4), (F32C, 100000, 200, 0.0, 4)])
def test_k_tiles_of_a_structure_factor_block(prec, n, P, skin, ktile):
    b = _batch([n], P, prec, skin=skin)
    assert R.rbsog_info(b.ctx)["rho_ktile"] == ktile
    b.close()


# the list build has the whole device where nothing runs beside it, where the
# evaluation builds for certain, and from 2^20 particles on
@pytest.mark.parametrize("prec,sizes,P,skin,wide", [
    (F32C, [100000], 500, None, 1), (F32C, [100000], 502, None, 0), (F64, [100000], 222, None, 0),
    (F32C, [100000], 502, 0.0, 1), (F32C, [2 ** 20 - 2], 60, None, 0), (F32C, [2 ** 20], 60, None, 1),
    (F32C, [2000] * 30, 10, None, 1)])
def test_grids_of_the_list_build(prec, sizes, P, skin, wide):
    b = _batch(sizes, P, prec, skin=skin)
    assert R.rbsog_debug_routes(b.ctx, False)["build_wide"] == 1
    assert _routes(b)["build_wide"] == wide


# two streams from 0.3 of that with a zero-frequency mode term
@pytest.mark.parametrize("prec,n,P,streams", [(F32C, 100000, 150, 1), (F32C, 100000, 151, 2), (F64, 60000, 110, 1),
                                              (F64, 60000, 111, 2)])
def test_streams_with_zero_modes(prec, n, P, streams):
    r = _routes(_batch([n], P, prec, zero_mode=1))
    assert (r["streams"], r["shared"]) == (streams, 2 - streams)


@pytest.mark.parametrize("prec", [F64, F32C])
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("sizes,P", [([1000], 31), ([3070, 66, 9000], 40)])
def test_zero_modes_share_launches_like_other_batches(prec, mode, sizes, P):
    """With a zero-frequency mode term the launches are shared too; timed kernel by
    kernel, each has its own: the same sums, so the same bits."""
    out = []
    for timed in (0, 1):
        b = _batch(sizes, P, prec, zero_mode=mode, device_chains=8)
        r = R.rbsog_debug_routes(b.ctx)
        assert (r["streams"], r["shared"]) == (1, 1)
        R.rbsog_profile(b.ctx, timed)
        F, E = b.forces()
        b.step(11, 1e-4)
        out.append((F, E, *R.rbsog_get_state(b.ctx, b.n), R.rbsog_get_energy(b.ctx)))
        b.close()
    for x, y in zip(*out):
        np.testing.assert_array_equal(x, y)
