"""Inline assembly in the kernels keeps nothing it changes from the compiler."""
import glob
import os
import re

from paper_2405_12631_amd import build as B


def test_asm_leaves_m0_to_the_compiler():
    """A load into LDS takes its address from m0: as an operand, so that the compiler sets the register and
    keeps no value of its own there across the statement (it only warns of m0 in a clobber list)."""
    loads = 0
    for path in glob.glob(os.path.join(B.CSRC, "*")):
        if not path.endswith((".hip", ".h")):
            continue
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"\basm\s+(?:volatile\s*)?\((.*?)\);", text, flags=re.S):
            assert not re.search(r"\bs_\w+\s+m0\b", m.group(1)), (path, m.group(0))
            if re.search(r"\blds\b", m.group(1).split("::")[0]):
                loads += 1
                assert '"{m0}"' in m.group(1), (path, m.group(0))
    assert loads >= 1
