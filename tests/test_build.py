"""What the build decides for each kernel set, from the sets' list in kernels.h."""
import os

import pytest

from paper_2512_22219_amd import build as B


def test_level_and_spills_of_every_set():
    sets = B.variants()
    assert len(sets) == 13
    for v in sets:
        assert v["level"] == ("-O3" if v["nb"] == 11 else "-Os"), v     # one packed row
        if v["nb"] in (1, 11, 4, 8, 16):                               # one row with two buffers, matrix cores
            assert v["spills"] == v["hybrid_spills"] == 0, v


REMARKS = """k.h:1:1: remark: Function Name: _ZN3mpk15mpk_mega_kernelILi2ELb1ELb0ELb0EEEvNS_8StepArgsE [-Rpass-analysis=kernel-resource-usage]
k.h:1:1: remark:     SGPRs Spill: 171 [-Rpass-analysis=kernel-resource-usage]
k.h:1:1: remark:     VGPRs Spill: %d [-Rpass-analysis=kernel-resource-usage]
k.h:1:1: remark: Function Name: _ZN3mpk15mpk_mega_kernelILi2ELb1ELb1ELb0EEEvNS_8StepArgsE [-Rpass-analysis=kernel-resource-usage]
k.h:1:1: remark:     VGPRs Spill: %d [-Rpass-analysis=kernel-resource-usage]
"""


def test_more_spills_than_recorded_fail_the_build():
    v = dict(index=7, nb=2, moe=True, level="-Os", spills=4, hybrid_spills=34)
    B.check_spills(v, REMARKS % (4, 34))
    for spills in ((5, 34), (4, 35)):
        with pytest.raises(RuntimeError, match="spills"):
            B.check_spills(v, REMARKS % spills)
    with pytest.raises(RuntimeError):
        B.check_spills(v, "")


@pytest.mark.parametrize("newer,rebuild", [(None, False), ("build.py", True), ("kernels.h", True), ("variants.hip", True), ("mpk.h", True)])
def test_a_library_older_than_what_it_is_made_from_is_stale(monkeypatch, newer, rebuild):
    monkeypatch.setattr(os.path, "exists", lambda p: True)
    monkeypatch.setattr(os.path, "getmtime", lambda p: 2.0 if os.path.basename(p) == newer else 1.0)
    assert B.stale() == rebuild
