"""The checks of test_isa_hazards.py for the direct-unit instantiations of the tile loops, which are compiled from the
same bodies under their own names (single_*, direct_*, wide_*_kernel), and a count of all kernels that copy tiles, so
that a new name does not go unchecked."""
import re

import pytest

import test_isa_hazards as hazards

# kernel templates and their instantiations: head dimensions x ragged x general; the wide ones are for d = 128 alone
DIRECT = {
    "fm_fwd.hip": {"single_fwd_kernel": 8, "direct_fwd_kernel": 8, "wide_fwd_kernel": 4},
    "fm_bwd.hip": {"single_dq_kernel": 8, "direct_dq_kernel": 8, "wide_dq_kernel": 4,
                   "single_dkdv_kernel": 8, "direct_dkdv_kernel": 8},
}
QUEUED = {"fm_fwd.hip": 8, "fm_bwd.hip": 16}


@pytest.fixture(scope="module", params=sorted(DIRECT))
def source_and_assembly(request, tmp_path_factory):
    return request.param, hazards._assembly(str(tmp_path_factory.mktemp("isa")), request.param)


def test_direct_lds_window_register(source_and_assembly):
    source, asm = source_and_assembly
    for kernel, count in DIRECT[source].items():
        hazards.check_lds_window_register(asm, [kernel], count)


def test_every_kernel_that_copies_tiles_is_named(source_and_assembly):
    source, asm = source_and_assembly
    copying = [m.group(1) for m in re.finditer(r"^(\w+):.*?^\.Lfunc_end\d+:", asm, re.S | re.M)
               if "global_load_lds" in m.group(0)]
    assert len(copying) == sum(DIRECT[source].values()) + QUEUED[source], copying


def test_direct_dkdv_inline_asm_mfma_wait_states(source_and_assembly):
    source, asm = source_and_assembly
    if source == "fm_fwd.hip":
        return
    for kernel in ("single_dkdv_kernel", "direct_dkdv_kernel"):
        hazards.check_inline_asm_mfma_wait_states(asm, kernel)


# The tile copies take their base address from a pair of scalar registers inside inline assembly, which the compiler's own hazard
# handling does not look into.  A vector instruction that writes a scalar register (v_readfirstlane, v_cmp, v_readlane) must be
# five wait states ahead of a vector memory instruction that reads it, or the copy goes to another address.
WAIT_STATES = 5


def _scalars(text):
    regs = {int(x) for x in re.findall(r"\bs(\d+)\b", text)}
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs.update(range(int(lo), int(hi) + 1))
    return regs


def _effect(ins):
    """(wait states, scalar registers that a vector instruction writes, those that a scalar one does, those that a copy reads)"""
    nop = re.match(r"s_nop (\d+)", ins)
    name, _, operands = ins.partition(" ")
    written = _scalars(operands.split(",")[0])
    if name.startswith("v_"):
        if re.match(r"v_(add_co|sub_co|subrev_co|addc_co|subb_co|div_scale|mad_u64|mad_i64)", name):
            written |= _scalars(operands.split(",")[1])   # the carry
        return 1, written, (), ()
    if name.startswith("global_load_lds"):
        return 1, (), (), _scalars(operands)
    return int(nop.group(1)) + 1 if nop else 1, (), written if name.startswith("s_") else (), ()


def _copies_too_early(lines):
    """Copies that read a base whose last writer is a vector instruction fewer than WAIT_STATES earlier, over all paths."""
    blocks = hazards._blocks(lines)
    effects = [[(ins, *_effect(ins)) for ins in b["ins"]] for b in blocks]
    state, work, bad = {0: {}}, [0], set()   # of a block: wait states since the write of each register, under WAIT_STATES
    while work:
        k = work.pop()
        ages = dict(state[k])
        for ins, passed, by_vector, by_scalar, read in effects[k]:
            if read and any(r in ages for r in read):
                bad.add(ins)
            if ages:
                ages = {r: a + passed for r, a in ages.items() if a + passed < WAIT_STATES and r not in by_scalar}
            for r in by_vector:
                ages[r] = 0
        for t in blocks[k]["succ"]:
            old = state.get(t)
            new = dict(old or {})
            for r, a in ages.items():
                new[r] = min(a, new.get(r, WAIT_STATES))
            if old is None or new != old:
                state[t] = new
                work.append(t)
    return bad


def test_a_base_written_too_late_is_seen():
    body = "v_readfirstlane_b32 s4, v0|s_mov_b32 m0, s9|s_nop {}|global_load_lds_dwordx4 v1, s[4:5] offset:1024|s_endpgm"
    assert _copies_too_early(body.format(2).split("|")) and not _copies_too_early(body.format(3).split("|"))
    assert _copies_too_early(["v_cmp_lt_i32_e64 s[4:5], s1, v0", "s_cbranch_scc1 .LBB0_1", "s_nop 7", ".LBB0_1:",
                              "global_load_lds_dwordx4 v1, s[4:5]", "s_endpgm"])                     # over a branch
    assert not _copies_too_early(["v_readlane_b32 s4, v0, 3", "s_add_u32 s4, s4, s6", "global_load_lds_dwordx4 v1, s[4:5]", "s_endpgm"])


def test_no_copy_reads_its_base_too_early(source_and_assembly):
    for m in re.finditer(r"^(\w+):.*?^\.Lfunc_end\d+:", source_and_assembly[1], re.S | re.M):
        if "global_load_lds" in m.group(0):
            bad = _copies_too_early(m.group(0).split("\n")[1:])
            assert not bad, f"{m.group(1)}: {sorted(bad)[:3]}"
