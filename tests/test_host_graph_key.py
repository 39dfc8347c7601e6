"""A captured launch sequence (QSV_RUN_GRAPH) is replayed only while every device
block that it uses is still the call's own. Scratch blocks are kept by position
and freed when a later call needs a larger one in the same place, so another
program's call between two graph calls can take any one of them away.

On the recorder: no replay runs after a block of its capture was freed, and a
replay does run where none was."""
import pytest

from tests.host_runtime import record

NOISY = 'ctx.load(W.c1_program(seed=8), noise=True), {shots}, dict(depolarizing=0.05)'
DERIVED = ('ctx.load("OPENQASM 3.0; include \\"stdgates.inc\\"; input float[64] a; input float[64] b; qubit[4] q; '
           'bit[4] c; rx(a + 2 * b) q[0]; ry(a - b) q[1]; rz(a) q[2]; c = measure q;"), 16, dict(theta=[0.1, 0.2])')
PARAM = ('ctx.load("OPENQASM 3.0; include \\"stdgates.inc\\"; input float[64] a; qubit[2] q; bit[2] c; '
         'rx(a) q[0]; c = measure q;"), 50000, dict(theta=[0.1])')
PLAIN = 'ctx.load(W.c1_program(seed=5, n={n})), {shots}, dict()'

RUN = """
ctx = Context(0)
a, shots, kw = {a}
b, b_shots, b_kw = {b}
run = lambda: a.run_shots(shots, seed=1, graph=True, **kw)
run()
run()
first = [count("hipStreamBeginCapture"), count("hipGraphLaunch"), count("hipFree")]
b.run_shots(b_shots, seed=2, **b_kw)
moved = count("hipFree") > first[2]
run()
run()
result = dict(first=first[:2], moved=moved, captures=count("hipStreamBeginCapture"),
              replays=count("hipGraphLaunch"), stale=stub.stub_stale_replays())
"""


@pytest.mark.parametrize("a, b", [
    (NOISY.format(shots=1500), PLAIN.format(n=13, shots=900)),   # the marks of touched phases
    (NOISY.format(shots=64), PARAM),
    (DERIVED, PARAM),                                            # the derived angles
    (PLAIN.format(n=14, shots=8), PLAIN.format(n=15, shots=8)),  # states
    (PLAIN.format(n=10, shots=8), PLAIN.format(n=10, shots=80000)),
], ids=["noise_marks", "noise_marks_resident", "derived", "states", "results"])
def test_no_replay_uses_a_freed_block(tmp_path_factory, a, b):
    r = record(tmp_path_factory.getbasetemp(), RUN.format(a=a, b=b))
    assert r["first"] == [1, 2]  # (captured once, replayed)
    assert r["moved"]
    assert r["stale"] == 0
    assert r["captures"] == 2 and r["replays"] == 4


def test_replays_go_on_where_no_block_moves(tmp_path_factory):
    r = record(tmp_path_factory.getbasetemp(),
               RUN.format(a=NOISY.format(shots=64), b=PLAIN.format(n=6, shots=4)))
    assert r == dict(first=[1, 2], moved=False, captures=1, replays=4, stale=0)
