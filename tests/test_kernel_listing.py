"""Properties of the compiled kernels that the source relies on and that no
run on the GPU would reliably show, read from the compiler's own output for
kernels.hip (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_02483_amd import build

pytestmark = pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="hipcc not available")


def _device(tmp, name, *flags):
    """Device side of kernels.hip with the build's own flags: (text, messages)."""
    out = str(tmp / name)
    src = os.path.join(build.CSRC, "kernels.hip")
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-device-only", "-S", src, "-o", out, *flags] + build.COMMON +
                       build.DEVICE, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(out) as f:
        return f.read(), r.stderr


@pytest.fixture(scope="module")
def ir(tmp_path_factory):
    return _device(tmp_path_factory.mktemp("ir"), "kernels.ll", "-emit-llvm")[0]


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    return _device(tmp_path_factory.mktemp("asm"), "kernels.s")


def test_no_compiler_warnings(listing):
    """A warning on the kernels is a defect to be seen: none of them are
    expected (in particular none on what an asm statement may clobber)."""
    found = [line for line in listing[1].splitlines() if "warning:" in line and "--hip-link" not in line]
    assert not found, found[:5]


def test_executor_lds_is_one_object(ir):
    """The operand ring's transfers address LDS below 64 KB and the ring is
    exactly that large at T = 64, so it has to start at LDS address 0: the
    executor keeps everything in LDS in one object whose first member it is."""
    shared = set(re.findall(r"^@([\w.$]+) = .*addrspace\(3\) global", ir, re.M))

    def lds_objects(function):
        return {name: {g for g in re.findall(r"@([\w.$]+)", body) if g in shared}
                for name, body in re.findall(r"^define [^\n]*@(\w*" + function + r"\w*)\((.*?)^}", ir, re.M | re.S)}

    kernels = lds_objects("exec_kernel")
    assert len(kernels) == 8
    for name, used in kernels.items():
        assert len(used) == 1, (name, used)
    # the one task body that is a function has none of its own
    for name, used in lds_objects("task_update_block").items():
        assert used <= set().union(*kernels.values()), (name, used)
