"""No fused product of the node update is left to the compiler (no GPU).

The step kernels (single steps, check steps, captured steps) and the steps on LDS
tiles are compiled apart from each other, and a node must come out the same in all
of them.  Where a sum has two products, the compiler's choice of the one to contract
into a fused multiply-add depends on the code around it; the update therefore writes
its fused products out.  Both files of kernels are compiled for gfx950 with contraction
allowed (the library's setting) and forbidden: every step and tile kernel must come
out instruction for instruction the same.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1409_5929_amd", "csrc")


def _kernels(asm):
    out, cur = {}, None
    for line in open(asm):
        m = re.match(r"(_Z\w*(?:k_step|k_tile)\w*):", line)
        if m:
            cur = out.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None and re.match(r"\s+[a-z]+_", line):
            cur.append(line.split(";")[0].strip())
    return out


@pytest.mark.parametrize("source,count", [("lbm_axi.hip", 12), ("lbm_axi_s16.hip", 40)])
def test_contraction_changes_no_instruction_of_the_update(tmp_path, source, count):
    from paper_1409_5929_amd.build import HIPCC_FLAGS

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    asm, jobs = {}, []
    for mode in ("off", "fast-honor-pragmas"):
        asm[mode] = tmp_path / f"{mode}.s"
        jobs.append(subprocess.Popen([hipcc, *flags, f"-ffp-contract={mode}", "-I" + os.path.join(ROOT, "include"),
                                      "--offload-device-only", "-S", "-o", str(asm[mode]), os.path.join(CSRC, source)],
                                     stderr=subprocess.DEVNULL))
    assert [j.wait() for j in jobs] == [0, 0]
    off, fast = (_kernels(asm[m]) for m in ("off", "fast-honor-pragmas"))
    assert len(off) == count and all(len(v) > 100 for v in off.values())
    assert off.keys() == fast.keys()
    assert [k for k in off if off[k] != fast[k]] == []
