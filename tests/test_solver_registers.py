"""What the compiler makes of the Gram path's solver kernels: no spilled registers, and with 8 samples a thread
no more registers than three workgroups a CU leave (one-vs-one trainings are batched by how many fit)."""
import os
import re
import subprocess

import pytest

from paper_2311_14908_amd import build as B


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_gram_path_solvers_keep_their_registers(tmp_path):
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-x", "hip", "-c", os.path.join(B.CSRC, "smo.hip"), "-o",
                        str(tmp_path / "smo.o"), "-Rpass-analysis=kernel-resource-usage"], check=True,
                       capture_output=True, text=True)
    seen = {}
    for block in r.stderr.split("Function Name: ")[1:]:
        m = re.match(r"_ZN4svmx9smo_solveILi256ELi(\d+)ELb1ELi0ELb0ELb([01])E", block)
        if m:
            spill = int(re.search(r"VGPRs Spill: (\d+)", block)[1])
            seen[int(m[1]), m[2] == "1"] = (spill, int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", block)[1]))
    assert len(seen) == 10
    assert all(spill == 0 for spill, _ in seen.values()), seen
    assert seen[8, False][1] >= 3, seen
