"""Which requests of a batch the persistent kernel may run: it takes states of up to
12 qubits whole, so their plan's tiles have to be the whole state, and wider ones
tile by tile in register phases, which tiles below 4 bits do not have. Programs
planned otherwise (an explicit plan, or a tuned one) take the tile passes."""
import pytest

from tests.host_runtime import record


@pytest.mark.parametrize("n, tile_bits, persistent", [
    (12, 12, True), (12, 11, False), (12, 10, False), (5, 5, True), (5, 4, False), (3, 3, True), (3, 2, False),
    (13, 12, True), (13, 10, True), (13, 4, True), (13, 3, False)])
def test_route(tmp_path_factory, n, tile_bits, persistent):
    r = record(tmp_path_factory.getbasetemp(), f"""
ctx = Context(0)
p = ctx.load(W.c1_program(seed=3, n={n}, layers=3, sites=(1,)))
p.replan({tile_bits}, 1, 0.5)
ctx.run_batch([dict(prog=p, shots=3, seed=1)])
result = [count("k_persistent"), count("k_tile_pass")]
""")
    assert (r[0] > 0) == persistent and (r[1] > 0) == (not persistent)
