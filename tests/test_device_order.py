"""The order of LDS accesses between lanes of one wave has to be stated to the compiler: it sees one lane's addresses, and
nothing else keeps a lane's read behind another lane's write.  No GPU: looks at the compiler's input for the device."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2510_26730_amd import build as b


def device_functions(src):
    """name -> body of every device function of `src` as the front end hands it to the optimiser."""
    if not shutil.which(b.HIPCC):
        pytest.skip("no HIP compiler here")
    flags = [f for f in b.FLAGS if f not in ("-shared", "-fPIC", "-pthread")]
    ir = subprocess.run([b.HIPCC, *flags, "--cuda-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes",
                         "-o", "-", os.path.join(b.CSRC, src)], check=True, capture_output=True, text=True).stdout
    return {m.group(1): m.group(2) for m in re.finditer(r"^define [^\n]*?@([\w$.]+)\([^\n]*\{\n(.*?)^\}", ir, re.M | re.S)}


def test_distance_blocks_order_their_operand_exchange():
    """Each stage of the distance blocks passes operands between lanes through the wave's own LDS buffer: ordered after
    the writes and again before the next stage overwrites them."""
    kernels = {n: body for n, body in device_functions("ef_dist.hip").items() if "dist_block_kernel" in n}
    assert len(kernels) == 4      # blocks of 32 x 32 and 64 x 64, four and eight waves
    for name, body in kernels.items():
        assert body.count("wave_lds_sync") >= 2, name
