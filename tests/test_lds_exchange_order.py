"""Lanes of a wave that hand one another values through LDS: between a write and the reads that follow it there is a barrier, of the wave or
of the workgroup, which also keeps the compiler from moving the one past the other (it sees one lane's addresses, and may find them
distinct).  Looks at the assembly of the kernels, basic block by basic block."""
import os
import re
import subprocess

import pytest

from paper_2507_10392_amd import build

UNITS = ["attention_f32", "attention_mfma", "gemm_f32", "gemm_small"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")
    cmd = [build._hipcc(), *build.FLAGS, "--cuda-device-only", "-S"]
    runs = {u: subprocess.Popen([*cmd, os.path.join(build.CSRC, u + ".hip"), "-o", str(out / u)], stderr=subprocess.PIPE) for u in UNITS}
    for u, p in runs.items():
        err = p.communicate()[1]
        assert p.returncode == 0, err.decode()[-2000:]
    return {u: (out / u).read_text().splitlines() for u in UNITS}


@pytest.mark.parametrize("unit", UNITS)
def test_reads_stand_behind_a_barrier(assembly, unit):
    pending, found, reads = None, [], 0
    for n, line in enumerate(assembly[unit]):
        op = line.strip()
        if re.match(r"(_Z\S+|\.LBB\S+):|s_c?branch", op) or "; wave barrier" in op or op.startswith("s_barrier"):
            pending = None
        elif op.startswith("ds_write"):
            pending = n
        elif op.startswith("ds_read"):
            reads += 1
            if pending is not None:
                found.append((pending + 1, n + 1))
    assert reads > 0 and not found, found[:5]
