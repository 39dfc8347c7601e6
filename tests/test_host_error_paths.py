"""A call that fails on the way leaves no work of its own on the stream: the
pinned block that its copies read and write belongs to the context's next call,
and the caller's arrays to the caller. On the recorder, with every allocation
and every copy of a call failing in turn."""
import pytest

from tests.host_runtime import record

RUN = """
left = []
for k in range(200):
    ctx = Context(0)
    p = ctx.load({prog})
    if {warm}:
        p.run_shots({shots} // 4, seed=1, **{kw})
    stub.stub_fail(b"{call}", k)
    try:
        p.run_shots({shots}, seed=1, **{kw})
        stub.stub_fail(b"", -1)
        break
    except QsvError:
        left.append(stub.stub_pending())
    ctx.close()
result = dict(failed=len(left), left=left)
"""


@pytest.mark.parametrize("call", ["hipMalloc", "hipMemcpyAsync"])
@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("prog, shots, kw", [
    ("W.c3_program(seed=3, n=14)", 64, "dict(share=True, state_out=True)"),
    ("W.c1_program(seed=1)", 40, "dict(state_out=True)"),
    ("lower(W.c1_program(seed=1, n=13), noise=True)", 40, "dict(depolarizing=0.1)"),
], ids=["shared", "resident", "noisy"])
def test_a_failed_call_leaves_nothing_queued(tmp_path_factory, call, warm, prog, shots, kw):
    r = record(tmp_path_factory.getbasetemp(), RUN.format(call=call, warm=warm, prog=prog, shots=shots, kw=kw))
    assert r["failed"] >= 1 and r["left"] == [0] * r["failed"]
