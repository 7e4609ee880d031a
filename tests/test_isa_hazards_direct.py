"""The checks of test_isa_hazards.py for the direct-unit instantiations of the tile loops (direct_*_kernel), which are
compiled from the same sources under their own names."""
import re

import pytest

import test_isa_hazards as hazards


def _direct_kernels_renamed(tmp_path, source="fm_bwd.hip", assembly=hazards._assembly):
    """The source's assembly with each direct kernel under the name of its queued counterpart, which is dropped."""
    asm = assembly(tmp_path, source)
    asm = re.sub(r"_ZN2fm\d+(fwd|dq|dkdv)_kernel", r"_ZN2fm_queued_\1_kernel", asm)
    length = {"fwd": 10, "dq": 9, "dkdv": 11}
    return re.sub(r"_ZN2fm\d+direct_(fwd|dq|dkdv)_kernel", lambda m: f"_ZN2fm{length[m.group(1)]}{m.group(1)}_kernel", asm)


def test_direct_dkdv_inline_asm_mfma_wait_states(tmp_path, monkeypatch):
    monkeypatch.setattr(hazards, "_assembly", _direct_kernels_renamed)
    hazards.test_dkdv_inline_asm_mfma_wait_states(tmp_path)


@pytest.mark.parametrize("source", ["fm_fwd.hip", "fm_bwd.hip"])
def test_direct_lds_window_register(tmp_path, monkeypatch, source):
    monkeypatch.setattr(hazards, "_assembly", _direct_kernels_renamed)
    hazards.test_lds_window_register_is_written_only_by_the_copy_helpers(tmp_path, source)


def _single_kernels_renamed(tmp_path, source="fm_bwd.hip", assembly=hazards._assembly):
    """The same for the kernels of whole units without setup launches."""
    asm = assembly(tmp_path, source)
    asm = re.sub(r"_ZN2fm\d+(fwd|dq|dkdv)_kernel", r"_ZN2fm_queued_\1_kernel", asm)
    length = {"fwd": 10, "dq": 9, "dkdv": 11}
    return re.sub(r"_ZN2fm\d+single_(fwd|dq|dkdv)_kernel", lambda m: f"_ZN2fm{length[m.group(1)]}{m.group(1)}_kernel", asm)


def test_single_dkdv_inline_asm_mfma_wait_states(tmp_path, monkeypatch):
    monkeypatch.setattr(hazards, "_assembly", _single_kernels_renamed)
    hazards.test_dkdv_inline_asm_mfma_wait_states(tmp_path)
