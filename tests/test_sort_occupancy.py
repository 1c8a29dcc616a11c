"""The sort kernels as compiled (CPU): registers allow as many workgroups a CU as their LDS does, two
of the 64-bit LSD passes and up to three of the bucket kernel.  They wait on loads and barriers in turn,
and another workgroup fills the waits.  (The 32-bit LSD passes are faster at two than at three.)"""
import re
import subprocess

import pytest

from paper_2608_15785_amd import build

LDS_BYTES, SIMDS = 160 * 1024, 4


@pytest.fixture(scope="module")
def kernels():
    cmd = [build.hipcc(), *build.COMMON, "--cuda-device-only", "-S", "-o", "/dev/null",
           "-Rpass-analysis=kernel-resource-usage", f"{build.CSRC}/k_sort.hip"]
    text = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    rows = re.findall(r"Function Name: (\S+).*?Occupancy \[waves/SIMD\]: (\d+).*?LDS Size \[bytes/block\]: (\d+)", text, re.S)
    return {name: (int(occ), int(lds)) for name, occ, lds in rows}


@pytest.mark.parametrize("kernel,threads", [("k_radix_passIm.*9PassShapeILi8ELi512E.*Lb0E", 512),
                                            ("k_radix_pass.*9PassShapeILi(8|10)ELi1024E.*Lb0E", 1024),
                                            ("k_bucket_sort.*11BucketShapeILi512E", 512),
                                            ("k_bucket_sort.*11BucketShapeILi1024E", 1024)])
def test_registers_allow_what_the_lds_does(kernels, kernel, threads):
    found = {k: v for k, v in kernels.items() if re.search(kernel, k)}
    assert found, kernel
    for name, (waves, lds) in found.items():
        assert waves >= LDS_BYTES // lds * (threads // 64) // SIMDS, (name, waves, lds)
