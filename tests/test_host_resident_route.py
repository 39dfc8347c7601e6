"""Which shot calls run as one resident launch: complex64 states of 12 qubits
that go gate by gate up to 256 shots, every other state of up to 12 qubits at
any count (launches seen by the recorder)."""
import pytest

from tests.host_runtime import record


@pytest.mark.parametrize("prog, kw, shots, resident", [
    ("W.logic_program(31, 12)", "dict(complex64=True)", 256, True),
    ("W.logic_program(31, 12)", "dict(complex64=True)", 257, False),
    ("W.logic_program(31, 12)", "dict()", 257, True),
    ("W.logic_program(31, 11)", "dict(complex64=True)", 257, True),
    ("W.brickwork_program(seed=1, n=12, layers=6, final_measure=True)", "dict(complex64=True)", 257, True),
], ids=["lists_256", "lists_257", "double", "eleven", "dense"])
def test_route(tmp_path_factory, prog, kw, shots, resident):
    r = record(tmp_path_factory.getbasetemp(), f"""
ctx = Context(0)
ctx.load({prog}).run_shots({shots}, seed=1, **{kw})
result = [count("k_resident"), count("k_tile_pass")]
""")
    assert (r[0] == 1 and r[1] == 0) if resident else (r[0] == 0 and r[1] > 0)
