"""Edges of the diagonal tile's factorisation (16 x 16 blocks inside 64- or
32-wide tiles) and of the workgroup's table of bins."""
import numpy as np
import pytest

import synth
from tests.gpu_util import have_gpu, run_instance, tol

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="no GPU")]


@pytest.mark.parametrize("ts", [64, 32])
@pytest.mark.parametrize("col", [0, 1, 14, 15, 16, 31, 32, 47, 48, 62, 63, 64, 79, 80, 111, 112, 129])
def test_pivot_failure_at_block_edges(orc, col, ts):
    """A NaN column of T fails at its own pivot, whatever its place in a
    16-wide block, as the oracle reports it."""
    inst = synth.small(seed=91, m=160, n=130, n_k=3, n_theta=2)
    inst.T = inst.T.copy()
    inst.T[:, col] = np.nan
    print(f"gpu: NaN column {col} tile {ts}", flush=True)
    got, info = run_instance(inst, ts=ts)
    np.testing.assert_array_equal(info, [col + 1, col + 1])
    assert np.all(got == -np.inf)


@pytest.mark.parametrize("n_k", [1, 255, 256, 257, 300])
def test_more_bins_than_the_table(orc, n_k):
    """Bins below, at and beyond the 256 a workgroup keeps in LDS; a bad
    theta in the last bin is found."""
    inst = synth.small(seed=92, m=500, n=400, n_k=n_k, n_theta=3)
    th = inst.theta.copy()
    th[1, n_k - 1] = np.nan
    ref, rinfo = orc.loglike_instance(inst, theta=th)
    print(f"gpu: n_k={n_k}", flush=True)
    got, info = run_instance(inst, theta=th)
    np.testing.assert_array_equal(info, rinfo)
    ok = info == 0
    assert ok.tolist() == [True, False, True]
    got, ref = got[ok], ref[ok]
    assert np.all(np.abs(got - ref) <= np.minimum(tol(ref), 1e-10 * np.abs(ref)))


@pytest.mark.parametrize("ts", [64, 32])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 48, 49, 63, 64, 65, 97, 112, 113])
def test_padded_blocks_are_left_out(orc, n, ts):
    """The 16-wide blocks of the last tile that hold only padding are not
    eliminated: 0 (a whole 32-wide tile of padding) to 4 of them."""
    inst = synth.small(seed=93, m=2 * n + 20, n=n, n_k=1, n_theta=3)
    ref, rinfo = orc.loglike_instance(inst)
    print(f"gpu: n={n} tile {ts}", flush=True)
    got, info = run_instance(inst, ts=ts)
    np.testing.assert_array_equal(info, rinfo)
    assert np.all(np.abs(got - ref) <= np.minimum(tol(ref), 1e-10 * np.abs(ref)))
