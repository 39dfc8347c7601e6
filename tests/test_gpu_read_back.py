"""Results read back in one block: through the context's pinned memory, and past
64 MiB through pageable memory; histories of shared trajectories grouped by the
bytes that they were read back as. Each against the same shots in other calls,
bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_11599_amd import Context
    c = Context(0)
    yield c
    c.close()


def _same(a, b):
    for x, y in [(a.creg, b.creg), (a.record, b.record), (a.n_events, b.n_events), (a.shot_status, b.shot_status),
                 (a.record_prob, b.record_prob)]:
        assert np.array_equal(x, y)


def test_more_than_the_pinned_block_holds(ctx):
    """50000 shots with 1200 recorded bits (1414 bytes a shot, 67 MiB) and the same in
    two calls of 25000 (34 MiB), then a small call in the block that is left."""
    lines = ["OPENQASM 3.0;", 'include "stdgates.inc";', "qubit[5] q;", "bit[1200] c;"]
    lines += [f"h q[{i % 5}]; c[{i}] = measure q[{i % 5}];" for i in range(1200)]
    prog = ctx.load("\n".join(lines) + "\n")
    a = prog.run_shots(50000, seed=3)
    for s0 in (0, 25000):
        b = prog.run_shots(25000, seed=3, shot_offset=s0)
        assert np.array_equal(a.creg[s0:s0 + 25000], b.creg)
        assert np.array_equal(a.record[s0:s0 + 25000], b.record)
        assert np.array_equal(a.record_prob[s0:s0 + 25000], b.record_prob)
    c = prog.run_shots(3, seed=3)
    assert np.array_equal(a.creg[:3], c.creg) and np.array_equal(a.record[:3], c.record)


@pytest.mark.parametrize("n, shots", [(2, 1), (2, 2), (2, 3000), (7, 4097), (12, 300)])
def test_histories_of_shared_trajectories(ctx, n, shots):
    """From one history to nearly as many as shots (measurements of every qubit between
    layers, and a branch on them)."""
    src = W.c1_program(seed=n, n=n, layers=4, sites=(1, 2, 3))
    prog = ctx.load(src)
    _same(prog.run_shots(shots, seed=9, share=True), prog.run_shots(shots, seed=9))
    _same(prog.run_shots(shots, seed=9, share=True, readout_error=0.2, reset_error=0.1),
          prog.run_shots(shots, seed=9, readout_error=0.2, reset_error=0.1))
