"""Composed phase matrices of noisy shots at the edges of their launch (four batch
elements a workgroup: batches of 1, 3, 4, 5 and 9), on programs that have such
phases: 10 qubits, where resident shots read the clean matrix of a phase without
a Pauli, and 13 qubits, where it is copied. At the rate taken some phases of
every batch are touched and some are not. Every shot equals the oracle's: records
bit for bit, the trajectory probability to 1e-12."""
import numpy as np
import pytest

import workloads as W
from oracle import sim
from paper_2604_11599_amd import lower
from paper_2604_11599_amd.api import plan_inspect

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [10, 13])
@pytest.mark.parametrize("shots", [1, 3, 4, 5, 9])
def test_each_batch_element_has_its_own_matrices(n, shots):
    from paper_2604_11599_amd import Context
    src = W.c1_program(seed=31, n=n, layers=5, sites=(1, 3))
    assert plan_inspect(lower(src, noise=True)).n_dense_phases >= 8
    ctx = Context(0)
    try:
        r = ctx.load(src, noise=True).run_shots(shots, seed=9, depolarizing=0.02, state_out=True)
        for s in range(shots):
            o = sim.run_shot(src, seed=9, shot=s, depolarizing=0.02)
            assert min(abs(e[3] - e[4]) for e in o.events) > 1e-12
            assert list(r.bits()[s]) == o.cbits
            assert abs(r.record_prob[s] - o.record_prob) <= 1e-12
            if s == 0:
                assert np.max(np.abs(r.state - o.psi.reshape(-1))) < 1e-10
    finally:
        ctx.close()
