"""No fused product of the node update is left to the compiler (no GPU).

The step kernels (single steps, check steps, captured steps) and the steps on LDS
tiles are compiled apart from each other, and a node must come out the same in all
of them.  Where a sum has two products, the compiler's choice of the one to contract
into a fused multiply-add depends on the code around it; the update therefore writes
its fused products out.  Both files of kernels are compiled for gfx950 with contraction
allowed (the library's setting) and forbidden: every step and tile kernel must come
out instruction for instruction the same.  The same compilation shows the tile kernels'
registers.
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


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """Device assembly of both files of kernels, with contraction forbidden and as the library has it."""
    from paper_1409_5929_amd.build import HIPCC_FLAGS

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    d = tmp_path_factory.mktemp("asm")
    out, jobs = {}, []
    for source in ("lbm_axi.hip", "lbm_axi_s16.hip"):
        for mode in ("off", "fast-honor-pragmas"):
            out[source, mode] = d / f"{source}.{mode}.s"
            jobs.append(subprocess.Popen([hipcc, *flags, f"-ffp-contract={mode}", "-I" + os.path.join(ROOT, "include"),
                                          "--offload-device-only", "-S", "-o", str(out[source, mode]),
                                          os.path.join(CSRC, source)], stderr=subprocess.DEVNULL))
    assert [j.wait() for j in jobs] == [0] * 4
    return out


@pytest.mark.parametrize("source,count", [("lbm_axi.hip", 12), ("lbm_axi_s16.hip", 40)])
def test_contraction_changes_no_instruction_of_the_update(asm, source, count):
    off, fast = (_kernels(asm[source, m]) for m in ("off", "fast-honor-pragmas"))
    assert len(off) == count and all(len(v) > 100 for v in off.values())
    assert off.keys() == fast.keys()
    assert [k for k in off if off[k] != fast[k]] == []


@pytest.mark.parametrize("source,count", [("lbm_axi.hip", 2), ("lbm_axi_s16.hip", 4)])
def test_tile_kernels_fit_two_blocks_on_a_compute_unit(asm, source, count):
    """k_tile, every storage type, with and without wall lanes: no scratch, and at most 128
    VGPRs, so that two blocks of 512 threads share a compute unit."""
    text = open(asm[source, "fast-honor-pragmas"]).read()
    seen = 0
    for entry in text[text.index("amdhsa.kernels:"):].split("  - .")[1:]:
        if not re.search(r"\.name:\s+_Z\w*k_tile", entry):
            continue
        field = {k: int(v) for k, v in re.findall(r"\.(private_segment_fixed_size|vgpr_count|vgpr_spill_count):\s+(\d+)", entry)}
        assert field["private_segment_fixed_size"] == 0 and field["vgpr_spill_count"] == 0, entry
        assert 0 < field["vgpr_count"] <= 128, entry
        seen += 1
    assert seen == count
