"""The tiled GEMM issues its MFMAs as inline assembly with the
accumulators tied to AGPRs, so the compiler's own hazard handling does not see
them.  What the kernel relies on is checked in the assembly that this source
compiles to: inside the k loop nothing but MFMAs touches an AGPR, the
accumulators' zeros are not written right before the first MFMA, and after the
last one the pipeline drains before any accumulator is read."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2411_03519_amd import build as b


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (shutil.which(b.HIPCC) or os.path.exists(b.HIPCC)):
        pytest.skip("hipcc not found")
    out = str(tmp_path_factory.mktemp("isa") / "gemm.s")
    subprocess.run([b.HIPCC, *b.COMMON, *b.DEVICE, "-x", "hip", "--offload-device-only", "-S",
                    os.path.join(b.PKG, "csrc/kernels/gemm.hip"), "-o", out], check=True, capture_output=True)
    text = open(out).read()
    found = {}
    for m in re.finditer(r"^(_ZN5metro\w*gemm_tiled_kernel\w*):", text, re.M):
        body = text[m.end():text.index(".Lfunc_end", m.end())]
        found[m.group(1)] = [ln.split(";")[0].strip() for ln in body.split("\n")]
    assert found
    return found


def test_accumulators_stay_in_place(kernels):
    for name, lines in kernels.items():
        ops = [ln for ln in lines if re.match(r"[a-z]", ln)]
        mfma = [i for i, ln in enumerate(ops) if ln.startswith("v_mfma")]
        agpr = [i for i, ln in enumerate(ops) if re.search(r"\ba(\[\d|\d)", ln) and not ln.startswith("v_mfma")]
        inside = [ops[i] for i in agpr if mfma[0] <= i <= mfma[-1]]
        assert not inside, (name, inside[:4])
        for i in mfma:
            d, c = re.match(r"v_mfma\w+ (\S+), \S+, \S+, (\S+)", ops[i]).groups()
            assert d == c and d.startswith("a["), ops[i]
        # a zero written before the loop is at least 4 instructions old when an MFMA adds to it
        # (2 wait states would do)
        first = {}
        for i in reversed(mfma):
            lo, hi = map(int, re.match(r"v_mfma\w+ a\[(\d+):(\d+)\]", ops[i]).groups())
            first.update((r, i) for r in range(lo, hi + 1))
        for i in agpr:
            if i < mfma[0]:
                r = int(re.match(r"v_accvgpr_write_b32 a(\d+), 0$", ops[i]).group(1))
                assert first[r] - i >= 4, (name, ops[i])
        # no vector instruction writes an operand of one of the next two MFMAs' slots (2 wait states)
        for i in range(mfma[0], mfma[-1]):
            d = re.match(r"(?!v_mfma)v_\w+ v(?:\[(\d+):(\d+)\]|(\d+))", ops[i])
            if not d:
                continue
            lo, hi = int(d.group(1) or d.group(3)), int(d.group(2) or d.group(3))
            for ln in ops[i + 1:i + 3]:
                for a, b in re.findall(r" v\[(\d+):(\d+)\]", ln) if ln.startswith("v_mfma") else ():
                    assert hi < int(a) or lo > int(b), (name, ops[i], ln)
        after = min(i for i in agpr if i > mfma[-1])
        assert "s_nop 7" in ops[mfma[-1] + 1:after], (name, ops[mfma[-1]:after + 1])
