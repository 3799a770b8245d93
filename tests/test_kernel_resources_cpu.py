"""What the compiler says about the registers of the matrix kernels (no GPU needed): the contractions keep everything in
registers.  A spill in their main loop costs more than what the loop's variants gain, and nothing else shows it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.timeout(600)
def test_no_contraction_spills(tmp_path):
    from paper_2509_13232_amd import build
    r = subprocess.run([build._hipcc(), *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, "pg_fused.hip"), "-o", str(tmp_path / "pg_fused.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    scratch, name = {}, None
    for line in r.stderr.splitlines():
        if m := re.search(r"remark: .*Function Name: (\S+)", line):
            name = m[1]
        elif m := re.search(r"remark: .*ScratchSize \[bytes/lane\]: (\d+)", line):
            scratch[name] = int(m[1])
    contractions = {k: v for k, v in scratch.items() if "gemm_store_kernel" in k}
    assert len(contractions) >= 8 and not any(contractions.values()), contractions
