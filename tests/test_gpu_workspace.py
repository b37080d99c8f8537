"""Workspaces shared by calls of different sizes: every result is that of the same call made first."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_iterative_spectra_of_mixed_sizes_in_one_process():
    """12, 11, 12, 13, 12 qubits, 32 levels: the block solver exchanges its workspaces every
    iteration and hands them on to the next size, above and below."""
    from paper_1710_03431_amd.binding import Engine
    insts = {nq: W.ring_instance(nq, 40 + nq, n_grid=12, n_levels=32) for nq in (11, 12, 13)}
    keep = Engine(0)   # keeps the cache between the calls
    first = {}
    for nq in (12, 11, 12, 13, 12):
        eng = Engine(0)
        eng.set_instance(insts[nq])
        eng.precompute(12, 32, method="iterative")
        got = eng.get_tables(("E", "Gamma", "leak"))
        if nq not in first:
            first[nq] = got
        for k, v in got.items():
            assert np.isfinite(v).all()
            np.testing.assert_array_equal(v, first[nq][k])
    del keep


def test_idle_workspaces_go_back_on_request():
    """The matrices of 200 points of 256 states, H and Z alone 210 MB, are free again; the next
    precompute gives the same tables."""
    import torch
    from paper_1710_03431_amd import binding
    inst = W.ring_instance(8, 48, n_grid=200)
    eng = binding.Engine(0)
    eng.set_instance(inst)
    binding.release_workspaces(0)
    eng.precompute(inst.n_grid, inst.levels)
    a = eng.get_tables(("E", "Gamma"))
    idle = torch.cuda.mem_get_info(0)[0]
    binding.release_workspaces(0)
    assert torch.cuda.mem_get_info(0)[0] - idle >= 200 << 20
    eng.precompute(inst.n_grid, inst.levels)
    b = eng.get_tables(("E", "Gamma"))
    for k in a:
        np.testing.assert_array_equal(a[k], b[k])
    with pytest.raises(binding.AqtError):
        binding.release_workspaces(1 << 20)
