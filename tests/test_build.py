"""The build refuses kernels whose vector registers spill."""
import glob
import os
import re
import subprocess

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


def test_the_attention_of_heads_of_64_keeps_five_waves_to_a_simd(monkeypatch, tmp_path):
    """Heads of 64 on the kernel of heads of 128 (162 and 243 registers: three and two waves) were a sixth to a third slower."""
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    kernel = "_ZN3amx25attention_fused_64_kernelILi2EEEvPKh"
    assert build.oversized_kernels(REMARKS.replace("_Z5firstv", kernel) % 0) == [kernel + " (it takes 256, 96 at most)"]
    assert build.oversized_kernels(REMARKS.replace("_Z5firstv", kernel).replace("256", "96") % 0) == []
    compiled = build._compile("attention_64.hip")
    assert compiled[1] == 0 and compiled[4] == []
    monkeypatch.setattr(build, "REGISTERS", {"attention_fused_64_kernel": 80})
    assert len(build._compile("attention_64.hip")[4]) == 4  # the kernel of each scale format is there


def test_the_attention_stores_its_rows_without_an_exchange_for_each(tmp_path):
    """The exchanges between lanes left in a kernel are those of a tile's maximum and sum, twice for pairs of tiles: one in front
    of every row's stores, 32 more, waited out 16 trips in a row."""
    listing = str(tmp_path / "attention.s")
    flags = [f for f in build.FLAGS if not f.startswith("-Rpass")]
    subprocess.run(["hipcc"] + flags + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "attention.hip"), "-o", listing], check=True,
                   capture_output=True)
    count, name = {}, None
    for line in open(listing):
        if line.startswith("_ZN3amx22attention_fused_kernel"):
            name = line.split(":")[0]
        elif "ds_bpermute_b32" in line:
            count[name] = count.get(name, 0) + 1
    assert len(count) == 8 and max(count.values()) <= 4


def test_inline_assembly_names_the_m0_it_writes():
    """The compiler keeps values in m0 (the address of a direct-to-LDS load, an index): a statement that writes it must say so."""
    statements = [m.group(0) for f in glob.glob(os.path.join(build.CSRC, "*")) for m in re.finditer(r"asm volatile\([^;]*?\);", open(f).read(), re.S)]
    writing = [s for s in statements if re.search(r"s_mov_b32 m0", s)]
    assert writing and all('"m0"' in s.rsplit(":", 1)[1] for s in writing)
