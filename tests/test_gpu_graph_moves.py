"""Graph replays with another program's larger call between them, which takes
over scratch blocks that the captured sequence had used (see
test_host_graph_key.py): every replay gives the eager call's results bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

DERIVED = ('OPENQASM 3.0; include "stdgates.inc"; input float[64] a; input float[64] b; qubit[4] q; bit[4] c; '
           "rx(a + 2 * b) q[0]; ry(a - b) q[1]; rz(a) q[2]; cx q[0], q[3]; c = measure q;")
PARAM = ('OPENQASM 3.0; include "stdgates.inc"; input float[64] a; qubit[2] q; bit[2] c; rx(a) q[0]; c = measure q;')


@pytest.mark.parametrize("src, noise, shots, kw, b_src, b_shots, b_kw", [
    (W.c1_program(seed=8), True, 1500, dict(depolarizing=0.05), W.c1_program(seed=5, n=13), 900, {}),
    (W.c1_program(seed=8), True, 64, dict(depolarizing=0.05), PARAM, 50000, dict(theta=[0.1])),
    (DERIVED, False, 16, dict(theta=[0.3, -1.1]), PARAM, 50000, dict(theta=[0.1])),
], ids=["noise", "noise_resident", "derived"])
def test_replays_after_a_larger_call(src, noise, shots, kw, b_src, b_shots, b_kw):
    from paper_2604_11599_amd import Context
    ctx, ref = Context(0), Context(0)
    try:
        a, b, r = ctx.load(src, noise=noise), ctx.load(b_src), ref.load(src, noise=noise)
        for seed in (1, 2, 3, 4):
            g = a.run_shots(shots, seed=seed, graph=True, **kw)
            e = r.run_shots(shots, seed=seed, **kw)
            for x, y in [(g.creg, e.creg), (g.record, e.record), (g.record_prob, e.record_prob),
                         (g.n_events, e.n_events)]:
                assert np.array_equal(x, y)
            b.run_shots(b_shots << min(seed, 2), seed=seed, **b_kw)
    finally:
        ctx.close()
        ref.close()
