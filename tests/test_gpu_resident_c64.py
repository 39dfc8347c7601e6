"""complex64 states of 12 qubits gate by gate, resident up to 256 shots and in
launches per pass and site beyond: the shots that both run are equal bit for bit,
and equal to shared trajectories'."""
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


def _same(a, b, count):
    for x, y in [(a.creg, b.creg), (a.record, b.record), (a.n_events, b.n_events), (a.shot_status, b.shot_status),
                 (a.record_prob, b.record_prob)]:
        assert np.array_equal(x[:count], y[:count])
    assert np.array_equal(a.state, b.state)


@pytest.mark.parametrize("noisy", [False, True])
def test_complex64_gate_lists_of_twelve_qubits(ctx, noisy):
    src = W.logic_program(31, 12)
    prog, kw = ctx.load(src, noise=noisy), dict(depolarizing=0.02) if noisy else {}
    a = prog.run_shots(256, seed=5, state_out=True, complex64=True, **kw)
    b = prog.run_shots(257, seed=5, state_out=True, complex64=True, **kw)
    _same(a, b, 256)
    if not noisy:
        _same(b, prog.run_shots(257, seed=5, state_out=True, complex64=True, share=True), 257)
