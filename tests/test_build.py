"""The build refuses kernels whose vector registers spill."""
import pytest

from paper_2411_09909_amd import build

REMARKS = """\
In file included from a.hip:3:
./a.h:94:1: remark: Function Name: _Z5firstv [-Rpass-analysis=kernel-resource-usage]
   94 |     int64_t M) {
      | ^
./a.h:94:1: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]
./a.h:94:1: remark:     SGPRs Spill: 4 [-Rpass-analysis=kernel-resource-usage]
./a.h:94:1: remark:     VGPRs Spill: %d [-Rpass-analysis=kernel-resource-usage]
a.hip:9:1: remark: Function Name: _Z6secondv [-Rpass-analysis=kernel-resource-usage]
a.hip:9:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:12:3: warning: unused variable 'x' [-Wunused-variable]
   12 |   int x;
"""


def test_spilling_kernels_are_named_and_remarks_are_not_shown():
    assert build.spilling_kernels(REMARKS % 0) == []
    assert build.spilling_kernels(REMARKS % 7) == ["_Z5firstv"]
    assert build._diagnostics(REMARKS % 7) == "a.hip:12:3: warning: unused variable 'x' [-Wunused-variable]\n   12 |   int x;"


def test_a_spill_fails_the_build(monkeypatch):
    monkeypatch.setattr(build, "_compile", lambda src: (src, 0, "", src, ["_Z5firstv"] if src == "cast.hip" else []))
    with pytest.raises(RuntimeError, match="cast.hip: vector registers spill in _Z5firstv"):
        build.build(verbose=False)
