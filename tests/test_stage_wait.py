"""The stage loads of the split-fp16 kernels go straight to LDS, so no register tells the compiler when they
are done: the wait for them stands in the source, ahead of the barrier that lets the other waves read."""
import os
import re
import subprocess

import pytest

from paper_2311_14908_amd import build as B


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src", ["gram_split.hip", "predict.hip"])
def test_loads_to_lds_are_waited_for(src, tmp_path):
    asm = tmp_path / "out.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "-x", "hip", "--offload-device-only", "-S", os.path.join(B.CSRC, src), "-o",
                    str(asm)], check=True, capture_output=True)
    found = 0
    for body in re.split(r"^_Z\w+:", asm.read_text(), flags=re.M)[1:]:
        body = body.split(".Lfunc_end")[0]
        if "global_load_lds" not in body:
            continue
        found += 1
        assert re.search(r"#ASMSTART\s+s_waitcnt vmcnt\(0\)\s+;;#ASMEND\s+(s_waitcnt [^\n]*\s+)?s_barrier", body)
    assert found >= 1
