"""Register steps of complex64 all-dense passes at the edges of their range:
tiles of 2^10, 2^11 and 2^12 amplitudes that are the whole state, the first
width with several tiles, passes of one phase, of staged matrices, of more
matrices than are staged, and of more steps than two registers hold. The steps
are taken from four tiles per resident workgroup on (at most 2048 workgroups of
64 threads, 1024 of the others).

Tolerance as for every complex64 state: 2e-5 in the 2-norm against the
complex128 oracle (unit roundoff 6e-8, about 20 roundoffs per 16-term phase
product, a few dozen phases)."""
import numpy as np
import pytest

import workloads as W
from oracle import sim

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_11599_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [10, 11, 12, 13, 15])
@pytest.mark.parametrize("layers", [1, 3, 14])
def test_complex64_state_matches_oracle(ctx, n, layers):
    src = W.brickwork_program(seed=100 * n + layers, n=n, layers=layers)
    shots = 20000 if n == 10 else 10000 >> max(0, n - 12)
    got = ctx.load(src).run_shots(shots, state_out=True, complex64=True).state
    assert np.linalg.norm(got - sim.run_shot(src).psi) < 2e-5


@pytest.mark.parametrize("n", [11, 12, 14])
def test_complex64_collapse_and_flips_enter_the_next_pass(ctx, n):
    """Measurements and resets between dense passes: the pending collapse and
    the flip frame are applied when the next pass loads its tiles. Forced
    records, so that both precisions follow one trajectory."""
    src = W.c1_program(seed=n, n=n, layers=9, sites=(2, 4, 7), final_measure=False)
    forced = np.array([1, 0, 1], dtype=np.uint8)
    got = ctx.load(src).run_shots(10000 >> max(0, n - 12), seed=4, forced=forced, state_out=True, complex64=True)
    ref = sim.run_shot(src, seed=4, shot=0, forced=list(forced))
    assert list(got.bits()[0]) == ref.cbits
    assert abs(got.record_prob[0] / ref.record_prob - 1.0) < 4e-5
    assert np.linalg.norm(got.state - ref.psi) < 2e-5
