"""The programs of reg_step_programs.py launch the register-step kernel of
complex64 dense passes: with the pass's matrices staged in LDS and, where a pass
has more phases than that or every shot has matrices of its own, without; and
none of them runs resident. Steps beyond the eight that two registers hold."""
import pytest

from paper_2604_11599_amd.api import plan_inspect
from tests import reg_step_programs as P
from tests.host_runtime import record

RUN = """
from tests import reg_step_programs as P
ctx = Context(0)
ctx.load({src}, noise={noise}).run_shots({shots}, seed=1, complex64=True, **{kw})
result = [count("k_tile_pass_c64ILb1"), count("k_tile_pass_c64ILb0"), count("k_resident")]
"""


@pytest.mark.parametrize("n, layers", P.NARROW)
def test_narrow_tiles(tmp_path_factory, n, layers):
    st = plan_inspect(P.narrow(n, layers))
    staged, unstaged, resident = record(tmp_path_factory.getbasetemp(), RUN.format(
        src=f"P.narrow({n}, {layers})", noise=False, shots=P.NARROW_SHOTS[n], kw={}))
    assert resident == 0 and staged + unstaged == st.n_passes
    # the last pass of the long program has its layers from the third on: one phase a layer or more
    assert unstaged == (1 if layers == 24 else 0)
    assert layers != 24 or st.n_phases - 2 * (st.n_passes - 1) > 8


@pytest.mark.parametrize("n", P.NOISY)
def test_matrix_set_per_shot(tmp_path_factory, n):
    staged, unstaged, resident = record(tmp_path_factory.getbasetemp(), RUN.format(
        src=f"P.noisy({n})", noise=True, shots=P.NOISY_SHOTS[n], kw=dict(depolarizing=P.NOISY_RATE)))
    assert resident == 0 and staged == 0 and unstaged > 1
