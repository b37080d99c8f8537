"""One-wavefront tiles (up to 32 padded levels) against the FP64 oracle's trajectories on its own
tables, and their widths and remainders against each other."""
import numpy as np
import pytest

import workloads as W
from gpu_common import compare_jump_records, engine_with_oracle_tables
from oracle import spectrum, trajectories

pytestmark = pytest.mark.gpu


def _instance(nq, n_levels):
    # strong coupling and few grid points: several jumps per trajectory, some within one step
    return W.ring_instance(nq, 31 + nq, n_grid=41, t_f=60.0, eta=2e-2, n_levels=n_levels)


# padded level counts 16 and 32, full and partly filled; tiles of every width with a remainder
@pytest.mark.parametrize("nq,levels", [(1, 2), (3, 8), (4, 16), (5, 32), (6, 17), (6, 31)])
def test_trajectories_match_the_oracle(nq, levels):
    inst = _instance(nq, levels)
    tabs = spectrum.all_tables(inst)
    eng = engine_with_oracle_tables(inst, tabs)
    K = 45
    ref = trajectories.run(tabs, inst, K)
    assert max(len(j) for j in ref.jumps) > 5
    for tile in (8, 16, 32, 64):
        got = eng.run(K, "fp64", seed=inst.seed, instance_id=inst.instance_id, record_capacity=128, tile=tile)
        same, _ = compare_jump_records(got["jumps"], got["jump_count"], ref.jumps, inst.t_f)[:2]
        assert same == 1.0
        np.testing.assert_allclose(got["pgs_sum"], ref.pgs_sum, rtol=1e-9, atol=1e-9 * K)


# K at the ends of a tile, of the 8-trajectory range and beyond it
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("nq,levels", [(4, 16), (6, 32)])
def test_widths_agree(nq, levels, prec):
    from paper_1710_03431_amd.binding import Engine
    inst = _instance(nq, levels)
    eng = Engine(0)
    eng.set_instance(inst)
    eng.precompute(inst.n_grid, levels)
    for K in (1, 8, 63, 129, 16384, 16385 + 8):
        runs = [eng.run(K, prec, seed=3, record_capacity=8, final_state=True, tile=t) for t in (0, 8, 16, 32, 64)]
        for r in runs[1:]:
            for k in ("jump_count", "net_gs", "jump_totals", "net_hist", "final_state"):
                np.testing.assert_array_equal(r[k], runs[0][k])
            assert r["jumps"].tobytes() == runs[0]["jumps"].tobytes()
            # sums of K populations in [0, 1], grouped by 64 at most
            np.testing.assert_allclose(r["pgs_sum"], runs[0]["pgs_sum"], rtol=0, atol=64 * 2.3e-16 * K)
