"""What the source of the LayerNorm product has to guarantee about its loads of gain and shift, read from the assembly that the
compiler makes of it (CPU only)."""
import os
import re
import subprocess

import pytest

from paper_2412_11272_amd import build as B

SRC = os.path.join(B.CSRC, "gemm_small.hip")


def _kernels(tmp, extra=()):
    """name -> instructions of every instantiation of the kernel."""
    out = os.path.join(tmp, "listing.s")
    r = subprocess.run([B.HIPCC, *B._flags(SRC), *extra, "-S", "--offload-device-only", SRC, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels, name = {}, None
    for line in open(out):
        m = re.match(r"(_ZN\S*gemm_ln_kernel\S*):", line)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and re.match(r"\t[a-z]", line):
            kernels[name].append(line.strip())
    assert len(kernels) >= 18, sorted(kernels)         # three depths x 16 to 64 rows x two epilogues
    return kernels


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return _kernels(str(tmp_path_factory.mktemp("ln")))


def test_bounds_check_covers_the_whole_offset(built):
    """Rows shorter than 512 values: the loads of the second half reach past gain and shift and are cut off by the buffer's bounds
    check, which is defined for the vector offset; a scalar offset would be outside of it."""
    for name, ins in built.items():
        first = next(i for i in ins if i.startswith("buffer_load") and i.endswith("lds"))
        assert re.match(r"buffer_load_dwordx4 v\d+, s\[\d+:\d+\], 0 offen lds$", first), (name, first)
