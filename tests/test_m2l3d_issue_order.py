"""What the 3D contraction's wait for its LDS copies relies on, read from the
assembly that hipcc makes of it: in every instantiation the copies of an operator
are followed, before the barrier that hands it over, by at least as many loads
as the wait leaves outstanding, none of them a flat load (flat loads return out of
order with the copies); and the row of zeros that boxes outside the grid read lies
on 16 bytes, as the 16-byte loads of a row need."""
import os
import re
import subprocess

import pytest

from paper_2009_00767_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "m2l3d.s")
    subprocess.run([build.HIPCC] + build.COMMON +
                   ["--offload-device-only", "-S", os.path.join(build.CSRC, "m2l3d.hip"), "-o", out],
                   check=True, capture_output=True, timeout=300)
    with open(out) as f:
        return f.read()


def test_loads_behind_the_copies(assembly):
    kernels = re.findall(r"^_ZN\S*k_m2l3d_mfma\S*:.*?^\.Lfunc_end", assembly, re.S | re.M)
    assert len(kernels) == 34
    checked = 0
    for k in kernels:
        behind = waits = 0
        copied = False
        allowed = None
        for line in k.splitlines():
            op = line.split()[0] if line.split() else ""
            if op.startswith("flat_"):
                assert not copied, line
            if op.startswith("global_load_lds"):
                copied, behind, allowed = True, 0, None
            elif op.startswith("global_load"):
                behind += 1
            elif op == "s_waitcnt" and "vmcnt" in line:
                allowed = int(re.search(r"vmcnt\((\d+)\)", line).group(1))
            elif op == "s_barrier" and copied:
                assert allowed is not None and allowed <= behind, (k[:120], allowed, behind)
                waits += 1
                copied = False
        if "global_load_lds" in k:
            assert waits == 2  # the first operator and the loop's
            checked += 1
    assert checked == 32  # all but the FP64 operators of 125 point charges


def test_zero_row_alignment(assembly):
    m = re.search(r"\.p2align\s+(\d+)[^\n]*\n_ZN\S*g_zero_row\S*:", assembly)
    assert m and int(m.group(1)) >= 4
