"""Launch shapes of the persistent and resident kernels are worked out once: a
process that serves many different small programs (widths, classical bits and
record lengths each need their own LDS) asks the runtime for no occupancy twice."""
from tests.host_runtime import record


def test_a_launch_shape_is_worked_out_once(tmp_path_factory):
    r = record(tmp_path_factory.getbasetemp(), """
ctx = Context(0)
progs = []
for n in range(1, 13):
    for k in range(4):  # 0, 512, 1024 and 1536 bytes of classical bits
        bits = f"bit[{64 * 64 * k}] x; " if k else ""
        text = f"OPENQASM 3.0; include 'stdgates.inc'; qubit[{n}] q; {bits}bit c; h q[0]; c = measure q[0];"
        progs.append(ctx.load(text.replace("'", '"')))
        if n >= 10:  # (matrix phases only: another build)
            progs.append(ctx.load(W.brickwork_program(1, n, 4, final_measure=True).replace("qubit[", bits + "qubit[")))
for layers in range(1, 9):  # (tile passes of as many phases, their matrices in LDS too)
    progs.append(ctx.load(W.brickwork_program(1, 14, layers)))
asked = []
for k in range(2):
    for p in progs:
        for c64 in (False, True):
            p.run_shots(2, seed=1, complex64=c64)
    asked.append(count("hipOccupancy"))
result = asked
""")
    assert r[0] > 64 and r[1] == r[0]
