"""What the compiled kernels hold that no run can show."""
import os
import re
import subprocess

import pytest

from paper_2410_17446_amd import build


@pytest.mark.slow
def test_weight_gradient_orders_its_lds_exchanges(tmp_path):
    """The lanes of a wave exchange each segment through LDS without a workgroup barrier, so both
    directions (stores before the fragments' reads, those before the next stores) need a wave
    barrier that the compiler moves nothing across; it leaves a mark in the assembly.  That a
    build without it orders them by luck, every run of it passes."""
    out = tmp_path / "unet.s"
    subprocess.run([build.hipcc(), *build.flags(), "--cuda-device-only", "-S", os.path.join(build.CSRC, "unet.hip"),
                    "-o", str(out)], check=True, capture_output=True)
    kernels = re.findall(r"^(\w*k_conv3_wgrad_mfma\w*):(.*?)\.end_amdhsa_kernel", out.read_text(), re.S | re.M)
    assert len(kernels) == 2  # vector and scalar loads
    for name, text in kernels:
        assert text.count("; wave barrier") >= 2, name
