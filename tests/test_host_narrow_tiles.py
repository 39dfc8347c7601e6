"""Plans on very narrow tiles: every pass's tile holds at most the asked number of
qubits (two where one is asked for and a gate has two) and all qubits of its
gates, whatever number of low qubits the options always hold."""
import pytest

import workloads as W
from paper_2604_11599_amd import lower
from paper_2604_11599_amd.api import plan_inspect


@pytest.mark.parametrize("tile_bits", [1, 2, 3, 4, 5, 6, 12])
@pytest.mark.parametrize("n", [2, 3, 5, 7, 13])
def test_tiles_hold_their_gates(n, tile_bits):
    for seed in (1, 2):
        lp = lower(W.random_dynamic_program(seed, n, n_ops=60, final_measure=True))
        st = plan_inspect(lp, tile_bits)
        gate = 0
        for k in range(st.n_steps):
            if st.step_kind[k] != 1:
                continue
            mask = st.step_mask[k]
            assert bin(mask).count("1") == min(n, max(2, tile_bits))
            for i in st.gate_instr[gate:gate + st.step_count[k]]:
                q = lp.instr[i]
                assert mask >> int(q["q0"]) & 1
                assert int(q["q1"]) == 0xFFFFFFFF or mask >> int(q["q1"]) & 1
            gate += st.step_count[k]
        assert gate == st.n_gates
