"""The deterministic prefixes of a batch's streamed requests run in rounds: step
k of every request in one launch for its gate passes and initialisations and one
for its control-only sites, however many requests there are, and split where a
launch would pass 2^20 workgroups. Launches counted on the recorder."""
import pytest

from tests.host_runtime import record

PROGRAMS = """
hdr = "OPENQASM 3.0; include 'stdgates.inc'; qubit[13] q; bit[13] c; bit[4] d;".replace("'", '"')
ry = "".join(f"ry(0.{i + 1}) q[{i}]; " for i in range(13))
control = hdr + "".join(f"d = {k}; if (d == {k % 2}) {{ " + ry + "} " for k in range(5)) + "c = measure q;"
init = hdr + "reset q; " + ry + "c = measure q;"
plain = hdr + ry + "c = measure q;"
ctx = Context(0)
"""


@pytest.mark.parametrize("name", ["control", "init", "plain"])
def test_launches_do_not_grow_with_the_requests(tmp_path_factory, name):
    r = record(tmp_path_factory.getbasetemp(), PROGRAMS + f"""
p = ctx.load({name})
result = []
for requests in (1, 2, 40):
    before = count("kernel")
    ctx.run_batch([{{"prog": p, "shots": 2, "seed": k}} for k in range(requests)])
    result.append(count("kernel") - before)
""")
    assert r[0] == r[1] == r[2] > 1


def test_rounds_are_split_at_a_launch_limit(tmp_path_factory):
    """40000 requests of 17 qubits, 32 workgroups a step each."""
    r = record(tmp_path_factory.getbasetemp(), PROGRAMS.replace("[13]", "[17]").replace("range(13)", "range(17)") + """
from paper_2604_11599_amd import plan_inspect
p, st = ctx.load(control), plan_inspect(control)
prefix = []
while not (st.step_kind[len(prefix)] == 2 and st.step_mask[len(prefix)]):
    prefix.append(st.step_kind[len(prefix)])
stub.stub_watch(b"k_pass_units")
ctx.run_batch([{"prog": p, "shots": 2, "seed": 1}] * 40000)
result = dict(prefix=prefix, sites=count("k_site_units"),
              grids=[stub.stub_grid(i) for i in range(100) if stub.stub_grid(i) >= 0])
""")
    assert r["prefix"].count(0) == 1 and r["prefix"].count(1) > 1 and r["prefix"].count(2) > 1
    steps = r["prefix"].count(0) + r["prefix"].count(1)
    assert r["grids"] == [1 << 20, 32 * 40000 - (1 << 20)] * steps
    assert r["sites"] == r["prefix"].count(2)
