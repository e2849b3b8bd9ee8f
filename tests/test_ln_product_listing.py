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


@pytest.mark.parametrize("extra", [(), ("-mllvm", "-amdgpu-sched-strategy=iterative-ilp")], ids=["as-built", "another-schedule"])
def test_gain_and_shift_have_landed_at_the_first_barrier(extra, built, tmp_path):
    """The first barrier hands gain and shift to the other waves.  Nothing waits for their loads as such: they are the first loads
    of the kernel, loads complete in order, and the rows loaded after them have arrived by then.  Both have to hold however the
    compiler orders the instructions; the second schedule used to issue rows ahead of them."""
    for name, ins in (built if not extra else _kernels(str(tmp_path), extra)).items():
        barrier = next(k for k, i in enumerate(ins) if i.startswith("s_barrier"))
        loads = [k for k, i in enumerate(ins) if re.match(r"(buffer|global|flat)_load_", i)]
        assert ins[loads[0]].endswith("lds"), (name, ins[loads[0]])
        assert not [i for i in ins[:barrier] if i.startswith("ds_read")], name
        if "ELi0EEEv" in name:                       # depth known at run time only: its rows are loaded behind branches
            continue
        issued = landed = 0
        for i in ins[:barrier]:
            issued += bool(re.match(r"(buffer|global|flat)_load_", i))
            wait = re.match(r"s_waitcnt .*?vmcnt\((\d+)\)", i)
            landed = max(landed, issued - int(wait.group(1))) if wait else landed
        assert landed >= 1, name
