"""The compiled split-BF16 Legendre kernels, built here from source: no buffer load runs in
a loop over the values of a scalar offset kept in vector registers, and the main loop of
alm2map (spin 2) does not start by waiting for every load in flight."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2208_10154_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: assembly lines} of k_leg_bf16.hip"""
    if not shutil.which(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("isa") / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-x", "hip",
                    os.path.join(build.CSRC, "k_leg_bf16.hip"), "-o", out], check=True, capture_output=True)
    found, name = {}, None
    with open(out) as fh:
        for line in fh:
            m = re.match(r"(_ZN3sht\w*k_\w*):", line)
            if m:
                name = m.group(1)
                found[name] = []
            elif line.startswith(".Lfunc_end"):
                name = None
            elif name and not line.lstrip().startswith(";"):
                found[name].append(line.strip())
    return found


def loops(lines):
    """(first, last) line of every backward branch"""
    at = {x.split(":")[0]: i for i, x in enumerate(lines) if x.startswith(".LBB")}
    for i, x in enumerate(lines):
        m = re.match(r"s_c?branch\S*\s+(\.LBB\w+)", x)
        if m and at[m.group(1)] < i:
            yield at[m.group(1)], i


def test_no_load_loops_over_scalar_offsets(kernels):
    assert len(kernels) > 20
    for name, lines in kernels.items():
        for i, j in loops(lines):
            if j - i < 16:  # the load, the compare and the branch back
                body = "\n".join(lines[i:j])
                assert not ("v_readfirstlane" in body and "buffer_load" in body), (name, body)


def test_alm2map_spin2_loop_head_waits_for_its_operands_only(kernels):
    seen = 0
    for name, lines in kernels.items():
        if "k_a2m_spin2_bf" not in name:
            continue
        main = max(((sum("v_mfma" in x for x in lines[i:j]), i - j, i, j) for i, j in loops(lines)))
        head = []
        for x in lines[main[2]:main[3]]:
            if x.startswith(("buffer_load", "global_load", "v_mfma")):
                break
            head.append(x)
        assert not any("vmcnt(0)" in x for x in head), (name, head)
        seen += 1
    assert seen == 9
