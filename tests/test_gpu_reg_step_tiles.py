"""Register steps of complex64 dense passes on tiles of 2^10, 2^11 and 2^12
amplitudes that are a whole state, and with a matrix set per shot
(reg_step_programs.py; test_host_reg_step_route.py sees them launch the kernel).

Forced records put every shot on one trajectory, and each shot is a work item of
its own: all of them have the same arithmetic, so their probabilities are equal
bit for bit, also those that a workgroup takes after its first. Shot 0 agrees
with the complex128 oracle as every complex64 state does: amplitudes to 2e-5 in
the 2-norm, probability to 4e-5.

With a matrix set per shot, calls of few shots take the pass with an LDS round
trip per phase, whose sums have the same order: every output is equal bit for
bit. Some shots of later work items agree with the oracle."""
import numpy as np
import pytest

from oracle import sim
from tests import reg_step_programs as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_11599_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n, layers", P.NARROW)
def test_whole_state_tiles(ctx, n, layers):
    src = P.narrow(n, layers)
    forced = np.array([1, 0], dtype=np.uint8)
    got = ctx.load(src).run_shots(P.NARROW_SHOTS[n], seed=4, forced=forced, state_out=True, complex64=True)
    ref = sim.run_shot(src, seed=4, shot=0, forced=list(forced))
    assert np.all(got.shot_status == 0)
    assert np.all(got.record_prob == got.record_prob[0])
    assert np.all(got.creg == got.creg[0])
    assert abs(got.record_prob[0] / ref.record_prob - 1.0) < 4e-5
    assert np.linalg.norm(got.state - ref.psi.reshape(-1)) < 2e-5


@pytest.mark.parametrize("n", P.NOISY)
def test_matrix_set_per_shot(ctx, n):
    src, shots = P.noisy(n), P.NOISY_SHOTS[n]
    prog = ctx.load(src, noise=True)
    got = prog.run_shots(shots, seed=6, depolarizing=P.NOISY_RATE, complex64=True)
    few = shots // 10
    for s0 in range(0, shots, few):
        part = prog.run_shots(min(few, shots - s0), seed=6, shot_offset=s0, depolarizing=P.NOISY_RATE, complex64=True)
        k = len(part.record_prob)
        for x, y in [(got.creg, part.creg), (got.record, part.record), (got.record_prob, part.record_prob),
                     (got.n_events, part.n_events)]:
            assert np.array_equal(x[s0:s0 + k], y)
    checked = 0
    for s in (0, 1, shots // 2, shots - 2, shots - 1):
        o = sim.run_shot(src, seed=6, shot=s, depolarizing=P.NOISY_RATE)
        if min(abs(e[3] - e[4]) for e in o.events) < 1e-4:
            continue
        assert list(got.bits()[s]) == o.cbits
        assert abs(got.record_prob[s] / o.record_prob - 1.0) < 4e-5
        checked += 1
    assert checked >= 3
