"""Batched decoding's host side under failures (no GPU): a join that fails at any point leaves no slot, page or table entry
behind; a step's tokens are taken whether they come at once, late or with the stream's end, and their absence is reported.  The
runtime is compiled for the host with made-up HIP calls and the sanitizers, see sanitize/batch_host_main.cpp."""
import os

import pytest

from tests.test_sanitizers_host import HIPCC, SAN, _run


def test_batch_bookkeeping_under_failures(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "batch_host")
    host = []
    for f in SAN:
        host += ["-Xarch_host", f]
    cmd = [HIPCC, "-x", "hip", "-O0", "-g", "-std=c++17", "--cuda-host-only", "-no-hip-rt", "-fuse-cuid=none"] + host + \
          [os.path.join("tests", "sanitize", "batch_host_main.cpp"), "-lpthread", "-o", exe]
    _run(cmd, exe, tmp_path)
