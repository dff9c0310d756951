"""The static checks over the ISA of the kernels with inline assembly (hipcc -S, no GPU): every load that
may be in flight has its registers left alone, and no inline-assembly instruction reads a scalar register
too soon behind the vector instruction that wrote it."""
import re

import pytest

from paper_1804_02941_amd import isa_checks as ic


def test_the_kernels_with_inline_assembly_pass_both_checks():
    assert ic.check_sources(verbose=True) == 0


HAZARD = """
_ZN3dab4demoEv:
	v_cmp_ge_f32_e64 s[10:11], v0, v1
	s_and_b64 s[8:9], s[6:7], s[10:11]
	v_cndmask_b32_e64 v0, 0, 1, s[8:9]
	v_cmp_ne_u32_e64 s[10:11], 0, v0
	{between}
	;;#ASMSTART
	v_writelane_b32 v131, s10, 59
	;;#ASMEND
	s_endpgm
.Lfunc_end0:
"""


def test_the_scalar_read_check_sees_a_lane_write_right_behind_the_compare():
    (name, lines), = ic.kernels(HAZARD.format(between="v_mul_f32_e32 v2, v3, v4"))
    assert len(ic.scalar_read_hazards(lines)) == 1                  # one instruction in between: one wait state
    (name, lines), = ic.kernels(HAZARD.format(between="s_nop 1"))
    assert ic.scalar_read_hazards(lines) == []


IN_FLIGHT = """
_ZN3dab4demoEv:
	;;#ASMSTART
	buffer_load_dword v5, v1, s[0:3], 0 offen
	;;#ASMEND
	;;#ASMSTART
	buffer_load_dword v6, v1, s[0:3], 0 offen
	;;#ASMEND
	s_waitcnt vmcnt({n})
	v_add_u32_e32 v7, v5, v5
	s_waitcnt vmcnt(0)
	s_endpgm
.Lfunc_end0:
"""


def test_the_in_flight_check_sees_a_use_before_the_wait():
    (name, lines), = ic.kernels(IN_FLIGHT.format(n=2))
    assert len(ic.loads_in_flight(lines)) == 1                      # vmcnt(2) leaves both loads pending
    (name, lines), = ic.kernels(IN_FLIGHT.format(n=1))
    assert ic.loads_in_flight(lines) == []                          # the older load has landed


def test_the_sort_kernels_at_their_64_register_allocation_read_no_register_before_it_is_written():
    assert ic.check_estimators_without_the_reserved_register(verbose=True) == 0


UNWRITTEN = """
_ZN3dab4demoEv:
	v_mov_b32_e32 v1, 0
	s_cbranch_scc1 .LBB0_2
	v_mov_b32_e32 v2, 1
.LBB0_2:
	v_mov_b32_dpp v1, v0 row_shr:1 row_mask:0xf bank_mask:0xf
	v_add_u32_e32 v3, v1, v2
	s_endpgm
.Lfunc_end0:
"""


def test_the_read_before_write_check_sees_a_register_set_on_one_path_only():
    (name, lines), = ic.kernels(UNWRITTEN)
    bad = ic.reads_before_any_write(lines)
    assert len(bad) == 1 and bad[0][2] == [2]                      # v2 is set only when the branch is not taken


@pytest.fixture(scope="module")
def direct_isa(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "direct.s")
    ic.compile_to_isa("direct.hip", out)
    return open(out).read()


def test_the_padded_block_kernels_hold_both_bursts_of_loads_like_the_plain_ones(direct_isa):
    """Each burst has registers of its own; a padded form with fewer registers than the plain one waits for one burst before it
    requests the next (seen with 56 and 72 registers instead of 88 and 104)."""
    regs = dict(re.findall(r"\.amdhsa_kernel \S*binconv_block_kernelI(\w+?)EEv.*?\.amdhsa_next_free_vgpr (\d+)", direct_isa, re.S))
    padded = [k for k in regs if re.match(r"Lb1ELb[01]ELi[24]E", k)]
    assert len(padded) == 8
    for k in padded:
        assert int(regs[k]) >= int(regs["Lb0E" + k[4:]]), k


def test_the_store_addresses_of_the_persistent_kernel_are_not_worked_out_again_for_every_store(direct_isa):
    """Scalar stores of the fp32 output (F not a multiple of four): the four offsets of a lane stay in registers.  (Seen otherwise:
    318 selects between the stores, each into a register that the store before still reads.)"""
    bodies = re.findall(r"^_ZN\S*binconv_direct_kernelILi\dELi\dELb[01]ELb0EE\S*:(.*?)\.end_amdhsa_kernel", direct_isa, re.S | re.M)
    assert len(bodies) == 12
    for b in bodies:
        stores = b[b.index("buffer_store_dword "):b.rindex("buffer_store_dword ")]
        assert not re.findall(r"v_cndmask_b32\S* v\d+, v", stores)


def test_the_input_of_the_weights_only_layer_is_read_with_checked_offsets(tmp_path):
    """The last channels of the last pixel may lie past the end of the input: a buffer load reads zeros there only where the vector
    offset says so, the scalar one (third operand) is no part of the check."""
    out = str(tmp_path / "wbin.s")
    ic.compile_to_isa("wbin.hip", out)
    loads = re.findall(r"buffer_load_dwordx4 \S+ (\S+), s\[\d+:\d+\], (\w+) offen", open(out).read())
    assert len(loads) > 50 and all(scalar == "0" for _, scalar in loads)
