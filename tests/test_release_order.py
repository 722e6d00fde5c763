"""The search publishes finished token sets to workgroups on other chiplets:
it writes its L2 back and then stores a count.  The count must not be stored
before the write-back has completed, which only the compiled code shows (the
compiler has left that wait out).  The HIP sources that publish are compiled
for gfx950 here and the instructions behind each L2 write-back are read."""
import os
import re
import subprocess

import pytest

from paper_1808_00687_amd.csrc import build as hip_build

# the search with its published counts: alone (the incremental lattice pass
# follows it) and with record workgroups in its launch
SOURCES = ["search_kernel.hip", "search_record_kernel.hip"]


def _unwaited(asm: str):
    """(write-backs, those whose next memory instruction comes before a wait for all vector memory operations)."""
    lines = [x.split(";")[0].strip() for x in asm.splitlines()]
    lines = [x for x in lines if x]
    found, bad = 0, []
    for i, x in enumerate(lines):
        if not x.startswith("buffer_wbl2"):
            continue
        found += 1
        for y in lines[i + 1:]:
            if y.startswith("s_waitcnt") and "vmcnt(0)" in y:
                break
            if re.match(r"(global|flat|buffer|s_endpgm|s_branch|s_cbranch|s_setpc)", y):
                bad.append(y)
                break
    return found, bad


def test_the_reader_of_the_instructions():
    ok = "buffer_wbl2 sc1\ns_waitcnt vmcnt(0) lgkmcnt(0)\nglobal_store_dword v0, v1, s[0:1] sc1\n"
    assert _unwaited(ok) == (1, [])
    early = "buffer_wbl2 sc1\ns_nop 3\nglobal_store_dword v5, v2, s[10:11] sc1\ns_waitcnt vmcnt(0)\n"
    assert _unwaited(early) == (1, ["global_store_dword v5, v2, s[10:11] sc1"])


@pytest.mark.parametrize("source", SOURCES)
def test_count_is_stored_after_the_write_back(source, tmp_path):
    if not os.path.exists(hip_build.HIPCC):
        pytest.skip("needs hipcc")
    out = tmp_path / "k.s"
    subprocess.run([hip_build.HIPCC, "-x", "hip", *hip_build.FLAGS, "--cuda-device-only", "-S",
                    os.path.join(hip_build.HERE, source), "-o", str(out)], check=True, capture_output=True)
    found, bad = _unwaited(out.read_text())
    assert found >= 2, "no published count in %s" % source
    assert not bad, bad
