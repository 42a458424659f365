"""Wait states inside the kernels' inline assembly.  The assembler puts what
is written there into the stream as it stands: where the compiler would insert
a wait state by itself, the text has to hold it.  gfx9 needs one between a
scalar write of M0 and a load that goes to LDS at the offset in M0."""

import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_04526_amd", "csrc")


def asm_texts():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            src = f.read()
        for m in re.finditer(r"\basm(?:\s+volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", src):
            text = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            yield os.path.basename(path), [ins.strip() for ins in re.split(r"\\n|;", text) if ins.strip(" \\t")]


def test_a_wait_state_between_m0_and_every_lds_load():
    loads = 0
    for name, ins in asm_texts():
        ins = [i.replace("\\t", "").strip() for i in ins]
        for at, i in enumerate(ins):
            if not re.search(r"\blds\b", i):
                continue
            loads += 1
            writes = [k for k in range(at) if re.match(r"s_\w+\s+m0\b", ins[k])]
            assert writes, f"{name}: {i}: M0 is written outside the block"
            between = ins[writes[-1] + 1:at]
            assert any(b.startswith("s_nop") for b in between), f"{name}: no wait state before {i}"
    assert loads > 0
