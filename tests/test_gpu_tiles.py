"""Automatic split of a run into launches of several tile widths (256 and 128 levels) against
one launch of 8-trajectory tiles: the width and the launch a trajectory falls into change
neither its path nor its state, and the observable sums agree to FP64 summation error."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engines():
    from paper_1710_03431_amd.binding import Engine
    out = {}
    for nq in (7, 8):
        inst = W.pm1_all_to_all(nq, 1007, n_grid=18, t_f=400.0, eta=1e-3)
        eng = Engine(0)
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, inst.levels)
        out[1 << nq] = eng
    return out


# column tiles of 8 per CU (256 CUs): 1, 2, 3 and the 2 + 3 of 10^4 trajectories, a remainder
# of one trajectory in the last tile of each, and more columns than one widest round
@pytest.mark.parametrize("levels", [256, 128])
@pytest.mark.parametrize("K", [1, 2041, 4096, 6001, 10000, 20489])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_launch_plan_matches_single_width(engines, levels, K, prec):
    eng = engines[levels]
    a = eng.run(K, prec, seed=5, record_capacity=4, final_state=True)
    b = eng.run(K, prec, seed=5, record_capacity=4, final_state=True, tile=8)
    assert int(a["jump_totals"].sum()) > 0 or K == 1
    for k in ("jump_count", "net_gs", "jump_totals", "net_hist"):
        np.testing.assert_array_equal(a[k], b[k])
    assert a["jumps"].tobytes() == b["jumps"].tobytes()
    np.testing.assert_array_equal(a["final_state"], b["final_state"])
    # K summands in [0, 1], tile sums of up to 64 of them: 64 eps K bounds either grouping
    tol = 64 * np.finfo(np.float64).eps * K
    np.testing.assert_allclose(a["pgs_sum"], b["pgs_sum"], rtol=0, atol=tol)
    np.testing.assert_allclose(a["pgs_sumsq"], b["pgs_sumsq"], rtol=0, atol=tol)


@pytest.mark.parametrize("tile", [24, 32])
def test_widths_of_the_plan_stay_refused_as_explicit_tiles(engines, tile):
    from paper_1710_03431_amd.binding import AqtError
    with pytest.raises(AqtError):
        engines[256].run(64, "fp64", tile=tile)
