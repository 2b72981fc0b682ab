"""The built kernels keep the distances that their inline-asm MFMAs need.

conv_pp issues its matrix instructions as inline assembly, so the compiler
does not know that a result may only be read (or copied) some wait states
after its MFMA.  The source keeps every other use of the accumulators behind
a wait; the compiler may still place register copies, so the instructions of
the library as built are checked."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin",
                       "llvm-objdump")
AGPR = re.compile(r"\ba(\d+|\[\d+:\d+\])")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions per kernel of libctc.so, in address order."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    so = shutil.copy(os.path.join(ROOT, "paper_2609_16742_amd", "libctc.so"), d)
    subprocess.run([OBJDUMP, "--offloading", so], check=True, cwd=d,
                   capture_output=True)
    obj = [f for f in os.listdir(d) if "amdgcn" in f]
    assert len(obj) == 1, obj
    out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn",
                          os.path.join(d, obj[0])], check=True,
                         capture_output=True, text=True).stdout
    fns, cur = {}, None
    for line in out.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:$", line)
        if m:
            cur = fns.setdefault(m.group(1), [])
        elif cur is not None and line.startswith("\t"):
            cur.append(line.split("//")[0].strip())
    return fns


@pytest.fixture(scope="module")
def code(kernels):
    """The kernels with such MFMAs."""
    return {n: ins for n, ins in kernels.items() if "conv_pp" in n}


def test_results_are_rounded_to_fp32_before_fp16(kernels):
    """v_fma_mixlo_f16 / mixhi round a multiply-add once, straight to fp16:
    the fused and the separate kernels only agree bit for bit if none uses
    them for its scale and shift."""
    assert any("conv_ir" in n for n in kernels) and any("conv_dma" in n for n in kernels)
    once = {n: s for n, ins in kernels.items() for s in ins
            if s.startswith(("v_fma_mixlo", "v_fma_mixhi"))}
    assert not once, once


def _regs(operand):
    """VGPRs and AGPRs of an operand, as a set of (file, number)."""
    m = re.match(r"([va])(?:(\d+)|\[(\d+):(\d+)\])$", operand.strip())
    if not m:
        return set()
    lo, hi = (m.group(2), m.group(2)) if m.group(2) else m.group(3, 4)
    return {(m.group(1), r) for r in range(int(lo), int(hi) + 1)}


def test_every_instance_is_checked(code):
    """conv_pp's instances by kind: a kernel added or lost shows here."""
    kinds = [re.search(r"conv_pp(r|32)?I", n).group(0) for n in code]
    assert {k: kinds.count(k) for k in kinds} == {
        "conv_ppI": 11, "conv_pprI": 8, "conv_pp32I": 2}, sorted(code)


def test_accumulators_of_inline_mfmas_are_touched_only_at_a_distance(code):
    for name, ins in code.items():
        waits = [i for i, s in enumerate(ins) if s == "s_nop 11"]
        assert len(waits) == 1, name
        # the loop up to the wait is one basic block
        top = max(i for i in range(waits[0]) if re.match("s_c?branch", ins[i]))
        mfma = [i for i in range(top, waits[0]) if ins[i].startswith("v_mfma")]
        uses = [i for i, s in enumerate(ins[:waits[0]])
                if AGPR.search(s) and not s.startswith("v_mfma")]
        assert len(mfma) >= 4 and "a[" in ins[mfma[0]], name
        # no MFMA outside the block whose end waits
        assert sum(s.startswith("v_mfma") for s in ins) == len(mfma), name
        near = [ins[i] for i in uses if i > mfma[0] - 8]
        # (zeroed accumulators: well ahead of the first MFMA)
        assert not near, (name, near[:5])


def test_operands_of_inline_mfmas_are_written_at_a_distance(code):
    """A vector instruction may write an operand of an MFMA two wait states
    before it at the latest (fragments come from LDS, behind a waitcnt)."""
    for name, ins in code.items():
        for i, s in enumerate(ins):
            if not s.startswith("v_mfma"):
                continue
            src = set().union(*(_regs(o) for o in s.split(None, 1)[1].split(",")[1:]))
            for p in ins[i - 2:i]:
                if p.startswith("v_") and not p.startswith("v_mfma"):
                    dst = _regs(p.split(None, 1)[1].split(",")[0])
                    assert not dst & src, (name, p, s)
