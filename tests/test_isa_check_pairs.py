"""The build's assembly check on scalar pairs spilled with one half
overwritten."""
import pytest

from paper_2304_05657_amd.isa_check import check_kernel

LOAD = "s_load_dwordx4 s[64:67], s[0:1], 0xf8"
SPILL = ["v_writelane_b32 v212, s64, 62", "v_writelane_b32 v212, s65, 63"]
BACK = ["v_readlane_b32 s8, v212, 62", "v_readlane_b32 s9, v212, 63"]
USE = ["global_load_dword v1, v2, s[8:9]", "s_endpgm"]


@pytest.mark.parametrize("body,bad", [
    ([LOAD, "s_mul_i32 s64, s4, 12"] + SPILL + BACK + USE, True),          # the low half
    ([LOAD, "s_mul_hi_u32 s65, s4, s5"] + SPILL + BACK + USE, True),       # the high half
    ([LOAD] + SPILL + ["s_mul_i32 s64, s4, 12"] + BACK + USE, False),      # after the spill
    ([LOAD, "s_add_u32 s64, s64, 16"] + SPILL + BACK + USE, False),        # a change of the value itself
    ([LOAD, "s_ashr_i32 s65, s64, 31"] + SPILL + BACK + USE, False),       # a sign extension
    ([LOAD, "s_mov_b64 s[64:65], s[2:3]"] + SPILL + BACK + USE, False),    # a new pair
    ([LOAD, "s_mul_i32 s64, s4, 12"] + SPILL + BACK + ["s_add_i32 s10, s8, s9", "s_endpgm"], False),  # two words
    (["s_load_dword s65, s[0:1], 0x8", "s_mul_i32 s64, s4, 12"] + SPILL + BACK + USE, False),  # not loaded as a pair
])
def test_half_overwritten_pair(body, bad):
    assert bool(check_kernel(body)) == bad


def test_lanes_stored_again():
    """A later store of the same lanes (a tuple whose halves are dead by then)
    is not what an earlier reload reads."""
    again = ["s_mul_i32 s64, s4, 12"] + SPILL + ["s_endpgm"]
    assert not check_kernel([LOAD] + SPILL + BACK + USE[:1] + again)
