"""Resident shots (states of up to 12 qubits, the whole program in one launch)
against the launches per pass and site that shared trajectories take, which do
the same arithmetic in the same order: every output is equal bit for bit. Widths
around the tile path's edges (below 4 qubits, gate lists below 10, matrix-core
phases from 10), sites with more events than are staged at a time, errors,
forced records, both amplitude types, and one width past the range."""
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


def _equal(prog, shots, **kw):
    a = prog.run_shots(shots, state_out=True, **kw)
    b = prog.run_shots(shots, state_out=True, share=True, **kw)
    for x, y in [(a.creg, b.creg), (a.record, b.record), (a.n_events, b.n_events), (a.shot_status, b.shot_status),
                 (a.record_prob, b.record_prob), (a.state, b.state)]:
        assert np.array_equal(x, y)
    return a


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 9, 10, 11, 12, 13])
def test_guarded_programs(ctx, n):
    for seed in (1, 2, 3):
        prog = ctx.load(W.logic_program(10 * n + seed, n, n_ops=30))
        _equal(prog, 9, seed=seed)
        _equal(prog, 9, seed=seed, complex64=True, readout_error=0.1, reset_error=0.2)


@pytest.mark.parametrize("n", [4, 8, 10, 11, 12])
def test_dense_layers_with_sites(ctx, n):
    prog = ctx.load(W.c1_program(seed=n, n=n, layers=6, sites=(1, 3)))
    a = _equal(prog, 33, seed=5)
    _equal(prog, 33, seed=5, complex64=True)
    _equal(prog, 5, seed=6, forced=a.record[:5])


def test_more_events_than_are_staged(ctx):
    """One measurement feeding 70 conditions and classical assignments."""
    lines = ["OPENQASM 3.0;", 'include "stdgates.inc";', "qubit[3] q;", "bit[70] c;", "h q[0];", "c[0] = measure q[0];"]
    lines += [f"if (c[{i}] == 1) {{ c[{i + 1}] = 1; }}" for i in range(69)]
    lines += ["if (c[69] == 1) { x q[1]; }", "c[1] = measure q[1];"]
    r = _equal(ctx.load("\n".join(lines) + "\n"), 40, seed=2)
    bits = r.bits()
    assert all(b[0] == b[1] == b[69] for b in bits) and 0 < sum(b[0] for b in bits) < 40


@pytest.mark.parametrize("n, shots", [(10, 1024), (10, 1025), (12, 256), (12, 257)])
def test_around_the_shots_that_are_resident_at_once(ctx, n, shots):
    """The build for few waves takes calls whose shots all fit the chip at once."""
    _equal(ctx.load(W.c1_program(seed=n, n=n, layers=4, sites=(1, 2))), shots, seed=8)
