"""Registers of kernels whose wavefronts per SIMD a launch counts on, as the
compiler reports them (no GPU)."""

import re
import subprocess

from paper_1710_08332_amd import build


def vgprs(source, kernel):
    r = subprocess.run([build.HIPCC] + build.HIP_FLAGS +
                       ["--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
                        f"{build.CSRC}/{source}", "-o", "/dev/null"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.search(rf"Function Name: \w*{kernel}\w* .*?\n.*?TotalSGPRs.*?\n?.*?VGPRs: (\d+)",
                      r.stderr, re.S)
    return int(found.group(1))


def test_one_launch_batch_keeps_five_wavefronts_per_simd():
    # 512 registers a lane and SIMD, in steps of 8: 5 wavefronts up to 96
    assert vgprs("batch.hip", "batch_one_launch_kernel") <= 96
