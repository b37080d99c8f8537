"""Dense eigensolver and table kernels at every matrix order they take in registers (2 to 256) and at
odd level counts: energies against LAPACK, the tables' own sums, orthogonality of the overlaps."""
import numpy as np
import pytest

import workloads as W
from oracle import model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,nq,levels", [("ring", q, 1 << q) for q in range(1, 9)]
                         + [("pm1", 4, 16), ("pm1", 7, 128), ("ring", 6, 17), ("ring", 7, 63), ("ring", 8, 65),
                            ("ring", 9, 33)])
def test_energies_and_table_sums(kind, nq, levels):
    from paper_1710_03431_amd.binding import Engine
    make = W.ring_instance if kind == "ring" else W.pm1_all_to_all
    M = 6
    inst = make(nq, 40 + nq, n_grid=M, n_levels=levels)
    eng = Engine(0)
    eng.set_instance(inst)
    eng.precompute(M, levels)
    t = eng.get_tables()
    eps = np.finfo(np.float64).eps
    for g in range(M):
        s = g / (M - 1)
        H = model.hamiltonian_dense(inst, s)
        ref = np.linalg.eigvalsh(H)
        # backward stable on both sides: a few N eps |H|
        np.testing.assert_allclose(t["E"][g], ref[:levels], rtol=0, atol=8 * (1 << nq) * eps * np.abs(ref).max())
        if g == 0:
            continue
        # Gamma adds R channel by channel, target by target: n_q n additions of positive terms
        np.testing.assert_allclose(t["Gamma"][g], t["R"][g].sum(axis=(0, 2)), rtol=nq * levels * eps, atol=0)
        # the omega = 0 element is gamma(0) z_bb^2
        g0 = 2 * np.pi * inst.eta * inst.T
        np.testing.assert_allclose(np.einsum("ibb->ib", t["R"][g]), g0 * t["zdiag"][g] ** 2, rtol=8 * eps, atol=0)
        if g >= 2:
            O = t["O"][g]
            np.testing.assert_allclose(O.T @ O, np.eye(levels), rtol=0, atol=64 * (1 << nq) * eps)
