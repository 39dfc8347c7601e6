"""Gate lists of resident shots below 10 qubits, in one run or phase by phase (one
run from 8 qubits, or up to 256 shots), over more phases than are staged at a
time, against the launches per pass and site of shared trajectories: every
output equal bit for bit."""
import numpy as np
import pytest

import workloads as W
from paper_2604_11599_amd.api import plan_inspect

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_11599_amd import Context
    c = Context(0)
    yield c
    c.close()


def _same(a, b, count):
    for x, y in [(a.creg, b.creg), (a.record, b.record), (a.n_events, b.n_events), (a.shot_status, b.shot_status),
                 (a.record_prob, b.record_prob)]:
        assert np.array_equal(x[:count], y[:count])
    assert np.array_equal(a.state, b.state)


@pytest.mark.parametrize("n", [2, 3, 4, 7, 8, 9])
@pytest.mark.parametrize("c64", [False, True])
def test_gate_lists_in_one_run_or_by_phase(ctx, n, c64):
    src = W.c1_program(seed=n, n=n, layers=120, sites=(100, 110))
    assert n < 8 or plan_inspect(src).n_phases > 100  # (a phase a layer or more: over 64 in the first pass)
    prog = ctx.load(src)
    runs = [prog.run_shots(k, seed=3, state_out=True, complex64=c64) for k in (1, 256, 257)]
    ref = prog.run_shots(257, seed=3, state_out=True, share=True, complex64=c64)
    for k, r in zip((1, 256, 257), runs):
        _same(r, ref, k)
