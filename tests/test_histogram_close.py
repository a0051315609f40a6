"""The closing step of the histogram kernels, read in the assembly of this repository's own
source.  A workgroup's ticket says that its additions to the bins are done, and one thread's fence
before the ticket waits for the additions of that thread's wave only (a barrier does not wait for
atomics without a result): the first wave has to have made them all."""
import os
import re
import subprocess

import pytest

from paper_1904_01197_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "tools.s")
    source = next(s for s in build.SOURCES if s.endswith("ndq_tools.hip"))
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.HIPCC_FLAGS +
                          ["-I", build.ROOT + "/include", "-I", build.CSRC, "--cuda-device-only", "-S", source,
                           "-o", out], stderr=subprocess.DEVNULL)
    text = open(out).read()
    return {m.group(1): m.group(0).splitlines()
            for m in re.finditer(r"^(_ZN3ndq\d+histogram\w*):.*?^\.Lfunc_end", text, re.S | re.M)}


def test_one_wave_makes_a_workgroups_additions_and_waits_for_them_before_the_ticket(kernels):
    assert len(kernels) == 8
    for name, lines in kernels.items():
        bins = 1 << int(re.search(r"ILi(\d)E", name).group(1))
        atomics = [i for i, line in enumerate(lines) if "global_atomic_add_x2" in line]
        # the additions to the bins return nothing; the ticket returns what it found (sc0)
        ticket = next(i for i in atomics if " sc0" in lines[i])
        additions = [i for i in atomics if i < ticket]
        # an instruction of one wave reaches 64 bins: fewer instructions would need more waves
        assert len(additions) == (bins + 63) // 64, name
        barriers = [i for i in range(additions[-1], ticket) if "s_barrier" in lines[i]]
        assert barriers and any(re.search(r"s_waitcnt.*vmcnt\(0\)", lines[i])
                                for i in range(barriers[-1], ticket)), name
