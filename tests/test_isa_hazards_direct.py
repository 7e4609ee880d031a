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
