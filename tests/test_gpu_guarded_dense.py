"""Phases whose gates share one guard run as composed matrices: passes under
one guard, passes of several, a guarded pass that comes first (it initialises
the state whatever its guard says), resident and tiled states, persistent
batches, against the oracle: records bit for bit, probabilities to 1e-12,
amplitudes to 1e-10 (complex128) as for every trajectory."""
import numpy as np
import pytest

from oracle import sim

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_11599_amd import Context
    c = Context(0)
    yield c
    c.close()


def _layer(rng, n, cx=True):
    s = "".join(f"U({rng.random() * 3:.6f}, {rng.random() * 3:.6f}, {rng.random() * 3:.6f}) q[{q}]; " for q in range(n))
    return s + "".join(f"cx q[{q}], q[{q + 1}]; " for q in range(0, n - 1, 2))


def _program(seed, n):
    rng = np.random.default_rng(seed)
    return "\n".join([
        "OPENQASM 3.0;", 'include "stdgates.inc";', f"qubit[{n}] q;", f"bit[{n + 2}] c;",
        f"if (c[0] == {seed % 2}) {{ {_layer(rng, n)} }}",
        _layer(rng, n), f"c[0] = measure q[{n // 2}];",
        f"if (c[0] == 1) {{ {_layer(rng, n)} {_layer(rng, n)} }}",
        f"c[1] = measure q[{n - 1}];",
        f"if (c[1] == 1) {{ {_layer(rng, n)} }} else {{ {_layer(rng, n)} }}", _layer(rng, n),
        f"if (c[0] == 0) {{ rx(0.3) q[1]; }}",
        "".join(f"c[{q + 2}] = measure q[{q}]; " for q in range(n))]) + "\n"


def _check(got, src, seed, shots, psi=None):
    bits = got.bits()
    for s in range(shots):
        o = sim.run_shot(src, seed=seed, shot=s)
        if min(abs(e[3] - e[4]) for e in o.events) < 1e-12:
            continue
        assert list(bits[s]) == o.cbits
        assert abs(got.record_prob[s] - o.record_prob) < 1e-12
        if s == 0 and psi is not None:
            assert np.max(np.abs(psi - o.psi.reshape(-1))) < 1e-10


@pytest.mark.parametrize("n", [9, 10, 12, 13, 14])
@pytest.mark.parametrize("seed", [2, 3])
def test_guarded_layers(ctx, n, seed):
    src = _program(seed, n)
    prog = ctx.load(src)
    a = prog.run_shots(6, seed=seed, state_out=True)
    _check(a, src, seed, 6, a.state)
    b = prog.run_shots(6, seed=seed, share=True)
    assert np.array_equal(a.creg, b.creg) and np.array_equal(a.record_prob, b.record_prob)
    _check(ctx.run_batch([{"prog": prog, "shots": 6, "seed": seed}])[0], src, seed, 6)
    c = prog.run_shots(6, seed=seed, complex64=True, forced=a.record, state_out=True)
    assert np.all(np.abs(c.record_prob / a.record_prob - 1.0) < 4e-5)
    assert np.linalg.norm(c.state - a.state) < 2e-5
