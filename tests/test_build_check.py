"""What the build refuses in the device code that the compiler makes."""
import pytest

from paper_1908_10396_amd.build import shifts_by_last_register

# {amount}: of the shift; {other}: the highest register in use beside it
KERNEL = """_Z1kPyi:
	s_barrier
	ds_read_b64 v[26:27], v23 offset:12672
	s_waitcnt lgkmcnt(0)
	{shift}
	v_mov_b32_e32 v{other}, 0
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("shift,other,refused", [
    ("v_lshlrev_b64 v[28:29], v47, -1", 46, True),
    ("v_lshrrev_b64 v[28:29], v47, v[26:27]", 40, True),
    ("v_ashrrev_i64 v[28:29], v47, v[26:27]", 3, True),
    ("v_lshl_add_u64 v[28:29], v[26:27], v47, v[2:3]", 46, True),
    ("v_lshlrev_b64 v[28:29], v47, -1 ; comment", 48, False),  # the allocation goes on
    ("v_lshlrev_b64 v[28:29], v46, -1", 47, False),
    ("v_lshlrev_b64 v[28:29], v46, -1", 45, False),            # v47 is allocated all the same
    ("v_lshlrev_b64 v[28:29], s47, -1", 46, False),
    ("v_lshlrev_b64 v[46:47], 3, v[46:47]", 20, False),
    ("v_lshl_add_u64 v[46:47], v[46:47], 0, s[2:3]", 20, False),
])
def test_64_bit_shifts_by_the_last_register(shift, other, refused):
    text = KERNEL.format(shift=shift, other=other)
    quiet = KERNEL.format(shift="s_nop 0", other=other).replace("_Z1k", "_Z1a")
    for asm in (text + quiet, quiet + text):
        assert shifts_by_last_register(asm.splitlines(True)) == (["_Z1kPyi"] if refused else [])
