"""Small batches up to 32 levels run in tiles of four trajectories, and say so."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# trajectory counts around the tile; every instance's last tile is ragged but the fourth's
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("nq,levels", [(4, 16), (6, 32)])
def test_reported_width_is_the_one_that_ran(nq, levels, prec):
    """The batch reports 4; asked for explicitly the same kernel runs (every output bit equal), and
    single runs in tiles of 4 and of 8 have the same paths."""
    from paper_1710_03431_amd.binding import Batch, Engine
    inst = W.ring_instance(nq, 31 + nq, n_grid=41, t_f=60.0, eta=2e-2, n_levels=levels)
    Ks = (1, 3, 5, 8, 129)
    engines = []
    for _ in Ks:
        eng = Engine(0)
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, levels)
        engines.append(eng)
    runs = [dict(n_traj=K, seed=3, instance_id=k, record_capacity=8) for k, K in enumerate(Ks)]
    outs = []
    for explicit in (False, True):
        b = Batch(engines, [dict(r, tile=t) for r, t in zip(runs, tiles)] if explicit else runs, precision=prec,
                  graph=True, autotune=True)
        tiles = b.tiles
        assert tiles == [4] * len(Ks)
        b.launch()
        outs.append(b.results())
        b.close()
    for k, (r, a, e) in enumerate(zip(runs, *outs)):
        for f in a:
            np.testing.assert_array_equal(a[f], e[f])
        one = [engines[k].run(r["n_traj"], prec, seed=3, instance_id=k, record_capacity=8, final_state=True, tile=t)
               for t in (4, 8)]
        for f in ("jump_count", "net_gs", "jump_totals", "net_hist", "final_state"):
            np.testing.assert_array_equal(one[0][f], one[1][f])
        assert one[0]["jumps"].tobytes() == one[1]["jumps"].tobytes()
        # sums of K populations in [0, 1], grouped by 8 at most
        np.testing.assert_allclose(one[0]["pgs_sum"], one[1]["pgs_sum"], rtol=0, atol=8 * 2.3e-16 * r["n_traj"])


def test_width_of_four_is_refused_above_32_levels():
    from paper_1710_03431_amd.binding import AQT_EINVAL, AqtError, Engine
    inst = W.ring_instance(6, 37, n_grid=11)
    eng = Engine(0)
    eng.set_instance(inst)
    eng.precompute(inst.n_grid, inst.levels)
    with pytest.raises(AqtError) as e:
        eng.run(64, "fp64", tile=4)
    assert e.value.status == AQT_EINVAL


def test_launches_around_larger_runs_of_the_members():
    """A member's own runs, larger and in flight beside the batch, leave its sums alone."""
    from paper_1710_03431_amd.binding import Batch, Engine
    import torch
    inst = W.ring_instance(5, 35, n_grid=101)
    engines = []
    for _ in range(2):
        eng = Engine(0, stream=torch.cuda.Stream())
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, inst.levels)
        engines.append(eng)
    torch.cuda.synchronize()
    b = Batch(engines, [dict(n_traj=500, seed=3, instance_id=k) for k in range(2)], precision="fp64", graph=True,
              autotune=False)
    b.launch()
    first = b.results()
    outs = engines[1].alloc_outputs(40000)
    torch.cuda.synchronize()
    for _ in range(3):
        b.launch()
        engines[1].run_into(outs, 40000, "fp64", seed=9)
    torch.cuda.synchronize()
    again = b.results()
    for x, y in zip(first, again):
        np.testing.assert_array_equal(x["pgs_sum"], y["pgs_sum"])
        np.testing.assert_array_equal(x["pgs_sumsq"], y["pgs_sumsq"])
        np.testing.assert_array_equal(4 * x["jump_totals"], y["jump_totals"])
