"""The matrix-core SpMM loads registers from inline assembly: its machine code is read for instructions
that name a register while a load into it may be in flight (the build does the same)."""
import pytest

from paper_2006_10901_amd import build, loads_in_flight


def listing(*code):
    """Disassembler lines of `code`, four bytes each; a branch's operand is its target's place in the list."""
    lines = []
    for i, text in enumerate(code):
        note = f"{4 * i:012X}: 00000000"
        if "branch" in text:
            op, place = text.split()
            text, note = f"{op} 0", note + f" <kernel+0x{4 * int(place):x}>"
        lines.append(f"\t{text}  // {note}")
    return lines


L0, L1 = "global_load_dwordx4 v[0:3], v8, s[0:1]", "global_load_dwordx4 v[4:7], v8, s[0:1]"


@pytest.mark.parametrize("code,bad", [
    ((L0, L1, "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v3", "s_waitcnt vmcnt(0)", "v_mov_b32 v9, v4", "s_endpgm"), []),
    ((L0, L1, "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v4", "s_endpgm"), ["v_mov_b32 v9, v4"]),              # read
    ((L0, "v_mov_b32 v2, 0", "s_endpgm"), ["v_mov_b32 v2, 0"]),                                            # given out again
    ((L0, "s_waitcnt lgkmcnt(0)", "v_accvgpr_write_b32 a1, v2", "s_endpgm"), ["v_accvgpr_write_b32 a1, v2"]),
    (("global_load_dword a5, v8, s[0:1]", "v_accvgpr_read_b32 v1, a5", "s_endpgm"), ["v_accvgpr_read_b32 v1, a5"]),
    # one path has a load less behind the first: vmcnt(1) is not enough there
    ((L0, "s_cbranch_scc1 3", L1, "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v0", "s_endpgm"), ["v_mov_b32 v9, v0"]),
    # a loop that waits for the load of the round before, and one that does not
    ((L0, L1, "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v0", L0, "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v4", "s_cbranch_scc0 1",
      "s_endpgm"), []),
    ((L0, L1, "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v0", L0, "v_mov_b32 v9, v4", "s_cbranch_scc0 1", "s_endpgm"),
     ["v_mov_b32 v9, v4"]),
    # a store counts too, and its operands are looked at
    ((L0, "global_store_dword v8, v9, s[0:1]", "s_waitcnt vmcnt(1)", "v_mov_b32 v9, v0", "s_endpgm"), []),
    ((L0, "global_store_dword v8, v1, s[0:1]", "s_endpgm"), ["global_store_dword v8, v1, s[0:1]"]),
])
def test_hazards_are_found(code, bad):
    assert loads_in_flight.hazards(listing(*code)) == bad


def test_built_library_names_no_register_with_a_load_in_flight():
    assert loads_in_flight.check(build.LIB_PATH) == 8       # one or two tiles, whole or by chunks, 32- or 16-bit indices


def test_a_wait_taken_out_is_found():
    name, (base, lines) = [kv for kv in loads_in_flight.disassembly(build.LIB_PATH).items() if "spmm_mfma_kernel" in kv[0]][0]
    assert not loads_in_flight.hazards(lines, base)
    waits = [i for i, line in enumerate(lines) if "s_waitcnt vmcnt(40)" in line]
    assert len(waits) == 6                                   # one for each set of rows of B
    shorter = list(lines)
    shorter[waits[2]] = shorter[waits[2]].replace("vmcnt(40)", "vmcnt(48)")
    assert loads_in_flight.hazards(shorter, base)
