"""Composed phase matrices at the edges of their launch: four batch elements a
workgroup, so batches of 1, 3, 4, 5 and 9. Every shot of a noisy program has
matrices of its own and equals the oracle's shot: records bit for bit, the
trajectory probability to 1e-12 (as for every complex128 trajectory)."""
import pytest

import workloads as W
from oracle import sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shots", [1, 3, 4, 5, 9])
def test_each_batch_element_has_its_own_matrices(shots):
    from paper_2604_11599_amd import Context
    src = W.c1_program(seed=31, n=8, layers=5, sites=(1, 3))
    ctx = Context(0)
    try:
        r = ctx.load(src, noise=True).run_shots(shots, seed=9, depolarizing=0.2)
        bits = r.bits()
        for s in range(shots):
            o = sim.run_shot(src, seed=9, shot=s, depolarizing=0.2)
            assert min(abs(e[3] - e[4]) for e in o.events) > 1e-12
            assert list(bits[s]) == o.cbits
            assert abs(r.record_prob[s] - o.record_prob) <= 1e-12
    finally:
        ctx.close()
