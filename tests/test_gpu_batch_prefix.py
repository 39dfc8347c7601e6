"""Prefixes of streamed batch requests that hold more than gate passes: programs
that start with a reset (an initialisation of its own), and classical assignments
and conditions between the passes before the first measurement, beside plain
ones in one batch, against the oracle: bits exactly, probabilities to 1e-12."""
import numpy as np
import pytest

from oracle import sim

pytestmark = pytest.mark.gpu


def _program(kind, n, seed):
    rng = np.random.default_rng(seed)
    layer = lambda: " ".join([f"U({rng.random() * 3:.6f}, {rng.random() * 3:.6f}, {rng.random() * 3:.6f}) q[{q}];"
                              for q in range(n)] + [f"cx q[{q}], q[{q + 1}];" for q in range(0, n - 1, 2)])
    s = f'OPENQASM 3.0; include "stdgates.inc"; qubit[{n}] q; bit[{n}] c; bit[3] d;\n'
    if kind == "init":
        s += f"reset q[{seed % n}];\n"
    if kind == "control":  # the assignment's value decides which gates run, twice before anything is measured
        for k in (seed % 8, (seed + 3) % 8):
            s += f"d = {k}; if (d == {k}) {{ {layer()} }} else {{ {layer()} }} d[0] = d[1] ^ d[2]; if (d[0]) x q[1];\n"
    return s + layer() + f"\nc[0] = measure q[{n // 2}]; if (c[0]) {{ {layer()} }}\nc = measure q;\n"


@pytest.mark.parametrize("n", [13, 15])
def test_prefix_steps_of_many_requests(n):
    from paper_2604_11599_amd import Context
    srcs = [_program(kind, n, 10 * k + i) for k in range(2) for i, kind in enumerate(("control", "init", "plain"))]
    ctx = Context(0)
    try:
        res = ctx.run_batch([{"prog": ctx.load(s), "shots": 3, "seed": 20 + k} for k, s in enumerate(srcs)])
        for k, (src, r) in enumerate(zip(srcs, res)):
            for s in range(3):
                o = sim.run_shot(src, seed=20 + k, shot=s)
                if min(abs(e[3] - e[4]) for e in o.events) < 1e-12:
                    continue
                assert list(r.bits()[s]) == o.cbits, (k, s)
                assert abs(r.record_prob[s] - o.record_prob) < 1e-12
    finally:
        ctx.close()
