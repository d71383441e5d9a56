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


def _vgprs(operand):
    m = re.match(r"[-|]*v\[(\d+):(\d+)\]", operand) or re.match(r"[-|]*v(\d+)()\b", operand)
    return set(range(int(m[1]), int(m[2] or m[1]) + 1)) if m else set()


def _operands(ins):
    args = ins.split(None, 1)[1] if " " in ins or "\t" in ins else ""
    return [_vgprs(x.strip()) for x in args.split(",")]


TRANS = ("v_rsq", "v_rcp", "v_sqrt", "v_exp", "v_log", "v_sin", "v_cos")


def dpp_hazards(text):
    """(DPP instructions, those whose operands are not safe to read): the
    compiler does not look into the asm statements that hold them, so it adds
    no wait states.  A DPP operand has to be written two wait states before;
    any operand one after a transcendental and 19 after an FP64 matrix
    instruction; and a matrix instruction reads the result of a DPP
    instruction two after it.  Only code after which control falls through is
    looked at: a label or a branch that close counts as unsafe."""
    code = [x.split(";")[0].strip() for x in text.splitlines()]
    code = [x for x in code if x and not x.startswith((".", "//")) or re.match(r"\.LBB\w+:", x)]
    count, bad = 0, []
    for i, ins in enumerate(code):
        dpp, mfma = "_dpp" in ins, ins.startswith("v_mfma")
        if not dpp and not mfma:
            continue
        count += dpp
        ops = _operands(ins)
        reads = set().union(*ops) if dpp else set().union(*ops[1:])
        states = 0
        for prev in reversed(code[max(0, i - 24):i]):
            if prev.endswith(":") or prev.startswith(("s_branch", "s_cbranch", "s_setpc", "s_swappc")):
                if dpp and states < 2:
                    bad.append((prev, ins))
                break
            if prev.startswith("s_nop"):
                states += int(prev.split()[1], 0) + 1
                continue
            if prev.startswith("v_") and not prev.startswith("v_cmp"):
                dst = _operands(prev)[0]
                if dpp and (dst & ops[1] and states < 2 or dst & reads and (
                        prev.startswith(TRANS) and states < 1 or prev.startswith("v_mfma") and states < 19)):
                    bad.append((prev, ins))
                if mfma and "_dpp" in prev and dst & reads and states < 2:
                    bad.append((prev, ins))
            states += 1
    return count, bad


def test_dpp_operands_are_ready(listing):
    count, bad = dpp_hazards(listing[0])
    assert count > 500 and not bad, (count, bad[:5])


@pytest.mark.parametrize("code,unsafe", [
    ("v_mul_f64 v[2:3], v[4:5], v[6:7]\n s_nop 1\n v_fmac_f64_dpp v[8:9], -v[2:3], v[2:3] row_newbcast:3", False),
    ("v_mul_f64 v[2:3], v[4:5], v[6:7]\n s_nop 0\n v_fmac_f64_dpp v[8:9], -v[2:3], v[2:3] row_newbcast:3", True),
    ("v_mov_b32_e32 v3, v12\n s_mov_b32 s0, 0\n v_fmac_f64_dpp v[8:9], -v[2:3], v[2:3] row_newbcast:3", True),
    ("v_add_f64 v[8:9], v[4:5], v[6:7]\n s_nop 0\n v_fmac_f64_dpp v[8:9], -v[2:3], v[2:3] row_newbcast:3", False),
    ("v_rsq_f64_e32 v[8:9], v[4:5]\n v_fmac_f64_dpp v[8:9], -v[2:3], v[2:3] row_newbcast:3", True),
    ("v_mfma_f64_16x16x4_f64 v[2:9], v[20:21], v[22:23], 0\n s_nop 7\n v_mov_b64_dpp v[10:11], v[2:3]", True),
    ("v_fmac_f64_dpp v[8:9], -v[2:3], v[2:3]\n v_mfma_f64_16x16x4_f64 v[30:37], v[8:9], v[22:23], 0", True),
    (".LBB0_1:\n s_nop 0\n v_mov_b64_dpp v[10:11], v[2:3] row_newbcast:3", True),
])
def test_dpp_check_sees_planted_hazards(code, unsafe):
    first = "s_nop 7\n s_nop 7\n s_nop 7\n"
    assert bool(dpp_hazards(first + code)[1]) == unsafe


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
