"""Direct loads to LDS take their LDS base from m0.  A block that writes m0 itself cannot tell the compiler so (the register
is reserved: a clobber of it is not honoured), and the compiler uses m0 too, for register indexes known only at run time.
So the base goes in as an operand that lives in m0, and no block writes it."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_02272_amd", "csrc")


def asm_blocks(text):
    for m in re.finditer(r"\basm\s+volatile\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(c, 0)
            i += 1
        yield text[m.end():i - 1]


def test_the_lds_base_is_an_operand():
    loads = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        if not path.endswith((".hip", ".h")):
            continue
        for block in asm_blocks(open(path).read()):
            code = block.split("::")[0]
            assert not re.search(r"\bm0\s*,", code), (os.path.basename(path), block)
            if "_load_lds_" in code:
                loads += 1
                assert '"{m0}"(' in block and block.rstrip().endswith('"memory"'), (os.path.basename(path), block)
                assert re.match(r'\s*"s_nop 0', code), (os.path.basename(path), block)      # wait state after the write
    assert loads >= 6
