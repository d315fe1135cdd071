"""The adjoint convolution's tap runs and window are LDS reads in every form of the
kernel (conv_adj.hip): an address that has lost its address space becomes a generic
load, which waits for global memory too (one output tile, n = 61: 0.57 ms where LDS
reads take 0.19).  Read off the compiler's assembly; no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_18863_amd import build


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="no hipcc")
def test_no_generic_memory_instructions(tmp_path):
    out = str(tmp_path / "conv_adj.s")
    subprocess.check_call([build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only",
                                                         os.path.join(build.CSRC, "conv_adj.hip"), "-o", out],
                          stderr=subprocess.DEVNULL)
    kernel, reads, generic = None, {}, {}
    for line in open(out):
        m = re.match(r"(_Z\w*k_conv_adj\w*):", line)
        if m:
            kernel = m.group(1)
            reads[kernel] = generic[kernel] = 0
        elif kernel and re.match(r"\s+ds_read", line):
            reads[kernel] += 1
        elif kernel and re.match(r"\s+flat_(load|store|atomic)", line):
            generic[kernel] += 1
        elif "s_endpgm" in line:
            kernel = None
    assert len(reads) >= 8 and all(reads.values())
    assert not any(generic.values()), {k: n for k, n in generic.items() if n}
