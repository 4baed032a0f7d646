"""The prefill projections wait for direct global-to-LDS loads by COUNT: s_waitcnt vmcnt(n) leaves the n youngest loads
of the wave in flight, so a wait is right only for the order in which the compiler issued the loads.  These tests
read the instructions of the built library (no GPU), replay every such kernel's loads and waits in that order, and ask at
each barrier that hands a ring stage over whether all of the wave's pieces of that stage have landed."""
import os
import re
import subprocess

import pytest

from paper_2604_23467_amd import build as hip_build

OBJDUMP = os.path.join(os.path.dirname(hip_build.HIPCC), "..", "llvm", "bin", "llvm-objdump")
TILE = re.compile(r"^[0-9a-f]+ <_Z14pf_tile_kernelILi(\d)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)EE")
GEMM = re.compile(r"^[0-9a-f]+ <_Z14pf_gemm_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)EE")
LABEL = re.compile(r"^(?:[0-9a-f]+ )?<(L\d+)>:")


def _listing(tmp):
    lib = hip_build.LIB
    assert os.path.exists(lib), "build the library first"
    os.symlink(lib, os.path.join(tmp, "libll.so"))
    subprocess.run([OBJDUMP, "--offloading", "libll.so"], cwd=tmp, check=True, stdout=subprocess.DEVNULL)
    obj = next(f for f in os.listdir(tmp) if f.endswith("gfx950"))
    out = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", obj], cwd=tmp, check=True,
                         stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout
    kernels, body = {TILE: {}, GEMM: {}}, None
    for line in out.splitlines():
        if re.match(r"^[0-9a-f]+ <_Z", line):
            body = None
            for name, found in kernels.items():
                m = name.match(line)
                if m:
                    body = found.setdefault(tuple(int(x) for x in m.groups()), [])
        elif body is not None and line.strip():
            body.append(line.split("//")[0].strip())
    return kernels


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    return _listing(str(tmp_path_factory.mktemp("listing")))


@pytest.fixture(scope="module")
def kernels(listing):
    assert len(listing[TILE]) >= 10
    return listing[TILE]


def replay(body, pieces_per_stage, handovers):
    """(landed, asked) at the first `handovers` barriers: how many of the wave's ring pieces are known to have landed
    there, and how many the stage handed over there needs.  Early exits are not taken, the K loop is."""
    at = {}
    for i, line in enumerate(body):
        m = LABEL.match(line)
        if m:
            at[m.group(1)] = i
    flight, issued, landed, out = [], 0, 0, []
    pc = steps = 0
    while len(out) < handovers:
        steps += 1
        assert steps < 200000 and pc < len(body), "the K loop was not found"
        line = body[pc]
        op = line.split()[0] if line else ""
        pc += 1
        if op.startswith(("buffer_load", "global_load")):
            piece = line.rstrip().endswith(" lds") or op.startswith("global_load_lds")
            issued += piece
            flight.append(issued if piece else 0)
        elif op.startswith(("buffer_store", "global_store", "flat_", "scratch_")):
            flight.append(0)
        elif op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", line)
            keep = int(m.group(1)) if m else len(flight)
            while len(flight) > keep:
                landed = max(landed, flight.pop(0))
        elif op == "s_barrier":
            out.append((landed, (len(out) + 1) * pieces_per_stage))
        elif op == "s_branch":
            pc = at[line.split()[1]]
        elif op.startswith("s_cbranch"):
            to = at[line.split()[1]]
            if to < pc:
                pc = to
        assert op != "s_endpgm", "left the kernel before the hand-overs"
    return out


def _stages(key, body, handovers):
    mode, wm, wk, mt, nb, s32, ns, once = key
    return replay(body, 2 * nb * s32 // 4, handovers)


def test_first_stage_has_landed_at_the_first_barrier(kernels):
    bad = []
    for key, body in kernels.items():
        landed, asked = _stages(key, body, 1)[0]
        if landed < asked:
            bad.append("pf_tile_kernel%s: %d of %d pieces" % (key, landed, asked))
    assert not bad, "\n".join(bad)


def test_every_stage_has_landed_when_it_is_handed_over(kernels):
    """Through the first rounds of the ring, where the prologue's loads are still counted, and on into its steady state."""
    bad = []
    for key, body in kernels.items():
        for i, (landed, asked) in enumerate(_stages(key, body, 2 * key[6] + 2)):
            if landed < asked:
                bad.append("pf_tile_kernel%s: stage %d handed over with %d of %d pieces" % (key, i, landed, asked))
    assert not bad, "\n".join(bad)


def test_row_major_gemm_hands_over_landed_slabs_only(listing):
    """Its first barrier stands in front of the ring; from the second on every barrier hands a slab over."""
    assert len(listing[GEMM]) >= 3
    bad = []
    for key, body in listing[GEMM].items():
        rows, stages, wm, wn, bk = key[:5]
        pieces = (rows + 256) * bk * 2 // 1024 // (wm * wn)
        for i, (landed, _) in enumerate(replay(body, pieces, 2 * stages + 3)):
            if landed < i * pieces:
                bad.append("pf_gemm_kernel%s: barrier %d with %d of %d pieces" % (key, i, landed, i * pieces))
    assert not bad, "\n".join(bad)
