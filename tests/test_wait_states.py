"""Wait states written by hand hold only if the compiler cannot move what they wait for behind them: each such statement of the attention kernels has the
registers it is about as operands.  A clobbered memory does not order register arithmetic.  No GPU needed."""
import os
import re

from paper_2411_15871_amd import build as B


def test_wait_states_name_their_registers():
    source = open(os.path.join(B.CSRC, "attn_bf16.hip")).read()
    statements = re.findall(r'asm(?: volatile)?\("s_nop[^;]*;', source)
    assert len(statements) >= 5
    for s in statements:
        assert re.search(r'"[+=]&?[va]"\(', s), s
