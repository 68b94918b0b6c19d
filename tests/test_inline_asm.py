"""Direct loads to LDS take their LDS base from m0.  The compiler uses m0 too, for register indexes known only at run time, so
a block that writes it has to say so; the register is reserved and a clobber of it is not honoured, but an output that lives
in it is.  Early, as the block reads its inputs after the write."""
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


def test_writes_of_m0_are_outputs():
    loads = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        if not path.endswith((".hip", ".h")):
            continue
        for block in asm_blocks(open(path).read()):
            code, *operands = re.split(r'"\s*:', block, maxsplit=1)
            if not re.search(r"\bm0\s*,|_load_lds_", code):
                continue
            loads += 1
            assert re.match(r'\s*"s_mov_b32 m0, %1\\n\\ts_nop 0', code), (os.path.basename(path), block)      # with a wait state
            assert operands and operands[0].lstrip().startswith('"=&{m0}"(') and '"memory"' in operands[0], (os.path.basename(path), block)
    assert loads >= 5
