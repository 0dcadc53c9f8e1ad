"""A load written in inline assembly has its result only after a wait that the compiler knows nothing of: it takes the output
registers as written when the statement ends and may copy them there.  In these sources such a load either writes LDS or is
waited for in its own statement (no GPU needed)."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_01438_amd", "csrc")


@pytest.mark.parametrize("source", ["band.hip", "shrink.hip", "fp32.hip", "generic.hip", "pool.hip"])
def test_asm_loads_into_registers_wait_in_their_own_statement(source):
    text = open(os.path.join(CSRC, source)).read()
    for m in re.finditer(r"asm\s+(?:volatile\s*)?\((.*?)\);", text, flags=re.S):
        statement = m.group(1)
        loads = [w for w in re.findall(r"\b(?:global|buffer|flat|ds|s)_(?:load|read)\w*", statement) if "_lds" not in w]
        assert not loads or "s_waitcnt" in statement, statement
