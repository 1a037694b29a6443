"""Registers of the de-dispersion's 16-wave kernels, from the compiler: a compute
unit holds one such work-group, 4 waves to a SIMD, and registers are handed out in
blocks of 8, so at more than 120 a wave nothing else (the copies and statistics
of another stream's chunk) can run beside it."""
import os
import re
import subprocess

import pytest

from paper_1611_09704_amd import build

CSRC = build.CSRC


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no HIP compiler")
def test_matrix_dedispersion_leaves_registers(tmp_path):
    out = str(tmp_path / "dedisp.s")
    subprocess.run([build.HIPCC] + build.CFLAGS + ["-S", "--cuda-device-only", os.path.join(CSRC, "spd_dedisp.hip"),
                                                   "-o", out], check=True, capture_output=True)
    found = re.findall(r"\.name:\s+\S*dedisp_mfma_kernelILi16E\S*(.*?)\.wavefront_size", open(out).read(), re.S)
    assert len(found) == 2
    for meta in found:
        assert int(re.search(r"\.vgpr_count:\s+(\d+)", meta).group(1)) <= 120
        assert int(re.search(r"\.vgpr_spill_count:\s+(\d+)", meta).group(1)) == 0
