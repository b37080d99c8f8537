"""Adjoint sweep against the oracle at 16 to 128 levels: the operand panels come in one, two or
four chunks of different lengths and the 16-byte tile copies leave part of the workgroup idle
below 128 levels.  (256 levels: test_gpu_grad.py.)"""
import numpy as np
import pytest

import workloads as W
from oracle import gradient

from gpu_common import compare_jump_records

pytestmark = pytest.mark.gpu

K = 17        # a ragged second tile


@pytest.fixture(scope="module")
def refs():
    A = np.array([2.0 * np.pi, np.pi, 2.5])
    B = np.array([0.6, np.pi, 2.0 * np.pi])
    out = {}
    for nq in (4, 5, 6, 7):
        inst = W.ring_instance(nq, 3, t_f=40.0, eta=2e-2, n_grid=12, A_ctrl=A, B_ctrl=B)
        out[nq] = (inst, gradient.trajectory_gradients(inst, K))
    return out


# FP64: the oracle's central differences (h = 1e-4) move by up to 1.3e-7 of their scale when h is
# halved, at 128 levels by 3.4e-6, so they are off by 4/3 of that; a margin of 4 and more.
# FP32: unit roundoff 6e-8 grown over 128-term sums, 11 steps and five products per step.
@pytest.mark.parametrize("segment", [0, 4])
@pytest.mark.parametrize("nq", [4, 5, 6, 7])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_per_trajectory_gradient(refs, nq, prec, segment):
    from paper_1710_03431_amd.binding import Engine
    inst, ref = refs[nq]
    eng = Engine(0)
    eng.set_instance(inst)
    eng.precompute(inst.n_grid, inst.levels)
    pt = eng.grad_pgs(K, prec, seed=inst.seed, instance_id=inst.instance_id, per_trajectory=True,
                      segment=segment)["per_traj"]
    P = pt.shape[1] // 2 - 1
    cap = max(len(j) for j in ref["jumps"]) + 1
    res = eng.run(K, prec, seed=inst.seed, instance_id=inst.instance_id, record_capacity=cap)
    rel = 1e-9 if prec == "fp64" else 1e-4
    same = [j for j in range(K)
            if compare_jump_records(res["jumps"][j:j + 1], res["jump_count"][j:j + 1], ref["jumps"][j:j + 1],
                                    inst.t_f, rel=rel)[0] == 1.0]
    assert len(same) >= (K if prec == "fp64" else K - 2), len(same)
    tol = 2e-4 if prec == "fp32" else (2e-5 if nq == 7 else 2e-6)
    for got, want in ((pt[same, 1:P + 1], ref["g"][same]), (pt[same, P + 2:], ref["score"][same])):
        scale = np.maximum(np.abs(want).max(axis=0), 1e-3)
        assert (np.abs(got - want) / scale).max() <= tol
