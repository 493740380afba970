"""What the compiler gives the whole-tile kernels of the bf16 path: their tile loops are laid out for two or more waves on a SIMD without a spill, and a
value too many that lives through them shows here first.  (Compiles for the GPU, runs nothing.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_07782_amd import build as b

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc here")
@pytest.mark.parametrize("source,kernels", [("bwd_bf16.hip", ("bwd_dkv8_bf16", "bwd_dkv_bf16", "bwd_dq_bf16", "bwd_dq_spill_bf16")),
                                            ("fwd_bf16.hip", ("fwd_bf16", "fwd_two_blocks_bf16"))])
def test_whole_tile_kernels_do_not_spill(source, kernels):
    cmd = [HIPCC] + b.FLAGS + b.EXTRA_FLAGS.get(source, []) + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                                                               os.path.join(b.CSRC, source), "-o", os.devnull]
    said = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", said, re.S)
    for k in kernels:
        scratch = {name: int(size) for name, size in found if f"{len(k) + 7}{k}_kernel" in name}
        assert scratch and not any(scratch.values()), scratch
