"""Registers, scratch and LDS of the kernels that stand in for the stage kernel,
as the compiler reports them under the library's own flags; CPU only.  What
their speed rests on: the wide kernel's population loop unrolled like the stage
kernel's, two split workgroups on a compute unit, and a resident kernel whose
few spilled registers stay few."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1702_01690_amd import build as B

LDS_PER_CU = 160 * 1024


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (metadata, body lines)"""
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
    out = tmp_path_factory.mktemp("asm") / "kernels.s"
    subprocess.run(["hipcc"] + flags + ["--offload-device-only", "-S", os.path.join(B.CSRC, "olb_kernels.hip"),
                                        "-o", str(out)], check=True, capture_output=True, timeout=900)
    text = out.read_text()
    got = {}
    for block in re.findall(r"  - \.agpr_count.*?\.wavefront_size: 64\n", text, flags=re.S):
        meta = dict(re.findall(r"^ *\.(\w+): +(\S+)$", block, flags=re.M))
        name = re.search(r"^    \.name: +(\S+)$", block, flags=re.M).group(1)
        start = text.index("\n" + name + ":")
        body = [line.strip() for line in text[start:text.index(".Lfunc_end", start)].split("\n")]
        got[name] = ({k: int(meta[k]) for k in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size",
                                               "group_segment_fixed_size")}, body)
    return got


def _of(kernels, name, count):
    got = {k: v for k, v in kernels.items() if name in k}
    assert len(got) == count, sorted(got)
    return got.items()


def test_wide_stage_kernels_are_unrolled(kernels):
    # {FP64, FP32} x walls x f^n
    for name, (meta, body) in _of(kernels, "wide_stage_kernelI", 8):
        assert sum(line.startswith("s_barrier") for line in body) == 25, name
        assert meta["private_segment_fixed_size"] == 0 and meta["vgpr_spill_count"] == 0, (name, meta)
        assert meta["vgpr_count"] <= (128 if "kernelId" in name else 80), (name, meta)


def test_two_split_workgroups_fit_a_compute_unit(kernels):
    # {FP64, FP32} x walls x f^n x specular x; twelve waves, three on each SIMD:
    # twice that at 80 registers
    for name, (meta, _) in _of(kernels, "split_stage_kernelI", 16):
        assert meta["private_segment_fixed_size"] == 0 and meta["vgpr_spill_count"] == 0, (name, meta)
        assert meta["vgpr_count"] <= 80 and 2 * meta["group_segment_fixed_size"] <= LDS_PER_CU, (name, meta)


def test_resident_kernels_keep_their_registers(kernels):
    # {FP64, FP32} x NG 1, 2, 3 x walls: 128 registers; only these three spill,
    # a handful of reloads a stage
    spills = {"kernelIdLi2ELb1E": 20, "kernelIdLi2ELb0E": 2, "kernelIdLi3ELb1E": 14}
    for name, (meta, _) in _of(kernels, "resident_kernelI", 12):
        most = next((n for k, n in spills.items() if k in name), 0)
        assert meta["vgpr_count"] <= 128 and meta["vgpr_spill_count"] <= most, (name, meta)
        assert meta["private_segment_fixed_size"] <= (36 if most else 0), (name, meta)
        assert meta["group_segment_fixed_size"] <= LDS_PER_CU
