"""The registers that the compiler gives the paired BLAKE3 compression's steps
(csrc/blake3.h), read from the assembly of this repository's own source: a step writes
its 16 state words before it reads the last of its message words, so no word may
share a register with the state, whatever the compiler knows of their values; and a
compression's last step leaves the wave at priority 0."""

import os
import re
import subprocess

import pytest

from paper_2607_01308_amd import build as B

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "paired_words.hip")


def _steps(asm):
    """The instruction lists of the step blocks of each kernel, in order."""
    kernels = re.split(r"\.globl\s+(\S+)", asm)[1:]
    for name, text in zip(kernels[::2], kernels[1::2]):
        steps = []
        for block in re.findall(r"#ASMSTART(.*?)#ASMEND", text, re.S):
            ins = [l.split(None, 1) for l in block.splitlines() if re.match(r"\s+[vs]_", l)]
            if any(op == "v_add3_u32" for op, _ in ins):
                steps.append([(op, [r.strip() for r in rest.split(",")]) for op, rest in ins])
        yield name, steps


def test_message_words_have_registers_of_their_own(tmp_path):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("needs the compiler")
    out = tmp_path / "paired.s"
    subprocess.run([hipcc, *B.COMMON, "-x", "hip", *B.DEVICE, "--cuda-device-only", "-S", SRC,
                    "-o", str(out)], check=True, capture_output=True)
    kernels = [(n, s) for n, s in _steps(out.read_text()) if s]
    assert len(kernels) == 4
    for name, steps in kernels:
        assert len(steps) == 14                     # two per round
        for step in steps:
            state = {r[0] for op, r in step if op.startswith("v_")}
            words = [r[3] for op, r in step if op == "v_add3_u32"]
            assert len(state) == 16 and len(words) == 8
            assert not state & set(words), name
        assert steps[-1][-1] == ("s_setprio", ["0"]), name
