"""CPU check of the instructions written by hand in inline assembly: the
compiler keeps the wait states between the instructions it emits, but none
inside an assembly block."""
import os
import re
import subprocess

import pytest

from paper_2604_25459_amd import build

SOURCES = [s for s in build.SOURCES
           if re.search(r'\basm\s*(volatile)?\s*\(\s*"[a-z]', open(os.path.join(build.CSRC, s)).read())]


def _sgprs(operand):
    """Scalar registers an operand names (vcc as "vcc")."""
    if operand == "vcc":
        return {"vcc"}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else set()


def _blocks(asm):
    return [[ln.split(";")[0].strip() for ln in b.splitlines() if ln.split(";")[0].strip()]
            for b in re.findall(r"#ASMSTART\n(.*?);;#ASMEND", asm, flags=re.S)]


@pytest.mark.parametrize("src", SOURCES)
def test_masks_written_and_read_by_vector_instructions_are_two_wait_states_apart(src, tmp_path):
    out = str(tmp_path / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, src), "-o", out],
                   check=True, capture_output=True)
    checked = 0
    for block in _blocks(open(out).read()):
        state, written = 0, {}              # wait states so far; register -> state after its last vector write
        for line in block:
            op, _, rest = line.partition(" ")
            args = re.findall(r"s\[\d+:\d+\]|[^,\s]+", rest)
            if op == "s_nop":
                state += int(args[0]) + 1
                continue
            state += 1
            if not op.startswith("v_"):
                continue
            # masks: the destination of a compare, the second one of an add or subtract with carry
            n_dst = 2 if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_", op) else 1
            for reg in set().union(*map(_sgprs, args[n_dst:])):
                if reg in written:
                    assert state - 1 - written[reg] >= 2, f"{src}: {reg} read too soon in\n" + "\n".join(block)
                    checked += 1
            for reg in set().union(*map(_sgprs, args[:n_dst])):
                written[reg] = state
    assert checked > 0
