"""The build's scan for hand-issued scalar loads: what it has to find, on assembly written here."""
import pytest

from paper_2506_11498_amd import build

LOAD = "\t;;#ASMSTART\n\t{}\n\t;;#ASMEND\n"
WAIT = "\t;;#ASMSTART\n\ts_waitcnt lgkmcnt(0)\n\t;;#ASMEND\n"
USE = "\ts_add_i32 s9, s8, 4\n"


@pytest.mark.parametrize("address", ["s[4:5], s6", "s[4:5], vcc_lo", "vcc, s6", "vcc, m0", "s[4:5], 0x10"])
def test_early_use_is_found_whatever_the_address_is_in(address):
    load = LOAD.format(f"s_load_dword s8, {address}")
    assert build._scan_scalar_loads(load + WAIT + USE, "x") == 1
    for early in (USE, "\tv_mov_b32_e32 v0, s8\n", "\ts_mov_b64 s[8:9], 0\n", "\ts_load_dwordx4 s[8:11], s[0:1], 0x0\n"):
        with pytest.raises(RuntimeError, match="s8 is touched"):
            build._scan_scalar_loads(load + early + WAIT, "x")


def test_loads_that_the_scan_cannot_judge_are_refused():
    for load in ("s_load_dword vcc_lo, s[4:5], s6", "s_load_dwordx2 s[8:9], s[4:5], s6"):
        with pytest.raises(RuntimeError, match="numbered register"):
            build._scan_scalar_loads(LOAD.format(load) + WAIT, "x")
    with pytest.raises(RuntimeError, match="never waited for"):
        build._scan_scalar_loads(LOAD.format("s_load_dword s8, s[4:5], s6"), "x")


def test_the_compilers_own_loads_are_left_alone():
    assert build._scan_scalar_loads("\ts_load_dword s8, s[4:5], s6\n" + USE + "\ts_waitcnt lgkmcnt(0)\n", "x") == 0
