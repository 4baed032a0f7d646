"""Registers and scratch of kernels that are built for a given number of waves per SIMD, from the metadata of the built
library (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2604_23467_amd import build as hip_build

LLVM = os.path.join(os.path.dirname(hip_build.HIPCC), "..", "llvm", "bin")


@pytest.fixture(scope="module")
def metadata(tmp_path_factory):
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("no llvm-readelf")
    tmp = str(tmp_path_factory.mktemp("notes"))
    os.symlink(hip_build.LIB, os.path.join(tmp, "libll.so"))
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "libll.so"], cwd=tmp, check=True,
                   stdout=subprocess.DEVNULL)
    obj = next(f for f in os.listdir(tmp) if f.endswith("gfx950"))
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], cwd=tmp, check=True,
                           stdout=subprocess.PIPE, text=True).stdout
    return {re.search(r"\.symbol:\s+(\S+)", k).group(1): k for k in re.split(r"\n  - ", notes) if ".symbol:" in k}


def _field(entry, name):
    return int(re.search(r"\.%s:\s+(\d+)" % name, entry).group(1))


def test_paged_attention_runs_four_waves_per_simd_without_scratch(metadata):
    found = {k: v for k, v in metadata.items() if "bt_attn_kernel" in k}
    assert len(found) == 4                                       # head_dim 64 and 128, 16 and 32 rows
    for name, entry in found.items():
        assert _field(entry, "vgpr_count") <= 128 and _field(entry, "private_segment_fixed_size") == 0, name


def test_one_workgroup_per_cu_kernels_keep_to_their_registers(metadata):
    """Two waves per SIMD at 512 threads a workgroup: 256 vector registers, and no scratch on the paths that wait for one
    another or stream the weights."""
    for part, count in (("decode_small_kernel", 4), ("pf_skinny_persist_kernel", 12)):
        found = {k: v for k, v in metadata.items() if part in k}
        assert len(found) == count
        for name, entry in found.items():
            assert _field(entry, "vgpr_count") <= 256 and _field(entry, "private_segment_fixed_size") == 0, name
