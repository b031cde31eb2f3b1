"""The reference encoders keep a block's texels in registers: no scratch, and no LDS (which a kernel that declares none
gets when the compiler moves an array there, and then addresses with values from the dispatch packet in host
memory).  From the compiler's report of the kernels' resources."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2407_09543_amd import build


def test_encoders_use_neither_scratch_nor_lds(tmp_path):
    if not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)):
        pytest.skip("needs hipcc")
    cmd = [build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                                         os.path.join(build.CSRC, "codec.hip"), "-o", str(tmp_path / "codec.o")]
    out = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    kernels = re.split(r"Function Name: ", out)[1:]
    seen = 0
    for k in kernels:
        if "k_encode_ref" in k.split()[0]:
            seen += 1
            use = {n: int(v) for n, v in re.findall(r"(ScratchSize|LDS Size) \[bytes/\w+\]: (\d+)", k)}
            assert use == {"ScratchSize": 0, "LDS Size": 0}, (k.split()[0], use)
    assert seen == 2
