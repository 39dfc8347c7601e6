"""Profiling events: where one cannot be made, the launch goes untimed and no
event handle of nothing is recorded (on the recorder, with the creation of every
event of a call failing in turn)."""
from tests.host_runtime import record


def test_no_event_is_recorded_that_was_not_made(tmp_path_factory):
    r = record(tmp_path_factory.getbasetemp(), """
ctx = Context(0, profile=True)
p = ctx.load(W.c1_program(seed=5, n=13))
q = [ctx.load(W.c3_program(seed=k, n=14, layers=2)) for k in range(2)]
failed = 0
for k in range(200):
    before = count("hipEventCreate")
    stub.stub_fail(b"hipEventCreate", 0)
    p.run_shots(2, seed=1)
    ctx.run_batch([{"prog": x, "shots": 4, "seed": 1} for x in q])
    if count("hipEventCreate") == before:
        break
    failed += 1
result = dict(failed=failed, empty=count("record of no event"), recorded=count("hipEventRecord"))
""")
    assert r["failed"] >= 4 and r["recorded"] > 0 and r["empty"] == 0
