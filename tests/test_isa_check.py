"""The build's assembly check on the join of a per-lane if without an else."""
import pytest

from paper_2304_05657_amd.isa_check import check_kernel

HEAD = ["s_and_saveexec_b64 s[2:3], vcc", "s_cbranch_execz .LBB0_2", "; %bb.1:", "v_mov_b32_e32 v7, 0", ".LBB0_2:"]
TAIL = ["s_or_b64 exec, exec, s[2:3]", "v_accvgpr_read_b32 v9, a4", "s_endpgm"]
COPY = "v_accvgpr_write_b32 a4, %s"


@pytest.mark.parametrize("body,bad", [
    (HEAD + [COPY % "v5"] + TAIL, True),                       # before EXEC is restored
    (HEAD + TAIL[:1] + [COPY % "v5"] + TAIL[1:], False),       # after it
    (HEAD + [COPY % "v7"] + TAIL, False),                      # a value of the then part
    (HEAD + [COPY % "v5"] + TAIL[:1] + TAIL[2:], False),       # never read
])
def test_copy_before_the_join(body, bad):
    assert bool(check_kernel(body)) == bad
