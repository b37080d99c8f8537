"""BF16 tiles that keep amplitudes as three BF16 words (64 levels and more): every tile width
gives the same paths and the same states as 8-trajectory tiles, and the states keep the FP32
bits that two words would lose."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engines():
    from paper_1710_03431_amd.binding import Engine
    out = {}
    for levels in (64, 100, 128):
        inst = W.pm1_all_to_all(7, 1007, n_grid=18, t_f=400.0, eta=1e-3)
        eng = Engine(0)
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, levels)
        out[levels] = eng
    return out


@pytest.mark.parametrize("levels,tile", [(64, 16), (64, 32), (64, 64), (100, 16), (100, 32), (100, 40),
                                         (128, 16), (128, 32), (128, 40)])
@pytest.mark.parametrize("K", [1, 63, 65])
def test_widths_agree(engines, levels, tile, K):
    eng = engines[levels]
    a = eng.run(K, "bf16", seed=5, record_capacity=4, final_state=True, tile=8)
    b = eng.run(K, "bf16", seed=5, record_capacity=4, final_state=True, tile=tile)
    for k in ("jump_count", "net_gs", "jump_totals", "net_hist"):
        np.testing.assert_array_equal(a[k], b[k])
    assert a["jumps"].tobytes() == b["jumps"].tobytes()
    np.testing.assert_array_equal(a["final_state"], b["final_state"])


def test_states_keep_fp32_precision(engines):
    # an FP32 mantissa has 24 bits, two words hold 16 of them: a state cut to two words would
    # leave the lowest 7 clear, one held in three has them set at random (1 in 128 clear)
    f = engines[128].run(512, "bf16", seed=5, final_state=True)["final_state"]
    f = f.reshape(512, -1)
    up = f.astype(np.float32).astype(np.float64)
    np.testing.assert_array_equal(f, up)       # amplitudes are FP32 values
    low = (f.view(np.uint64) >> np.uint64(29)) & np.uint64(0x7F)
    assert (low[f != 0] != 0).mean() > 0.9
