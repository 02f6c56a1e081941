"""Wide loads of tensors that the C ABI only promises at 4-byte alignment (router,
predictor factors, logits): the device code may read them several floats at a time
only through types declared at that alignment.  The hardware of this target takes a
16-byte load at any 4-byte address, so only the compiled code shows the difference:
no vector of floats may be loaded from global memory at a claimed alignment above 4."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_00395_amd import build as BLD

pytestmark = pytest.mark.skipif(shutil.which(BLD.HIPCC) is None, reason="hipcc not available")


# the sources whose float operands in global memory are the caller's, or doubles
@pytest.mark.parametrize("src", ["predictor.hip", "router.hip"])
def test_float_vectors_are_read_at_the_promised_alignment(src, tmp_path):
    out = str(tmp_path / "device.ll")
    subprocess.run([BLD.HIPCC, *BLD.FLAGS, "--cuda-device-only", "-emit-llvm", "-S",
                    os.path.join(BLD.CSRC, src), "-o", out], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    with open(out) as f:
        text = f.read()
    assert "amdgpu_kernel" in text
    loads = re.findall(r"load <\d+ x float>, ptr(?: addrspace\(1\))? [^\n]*?align (\d+)", text)
    too_wide = [a for a in loads if int(a) > 4]
    assert not too_wide, f"{len(too_wide)} of {len(loads)} float vector loads claim more than 4 bytes"
