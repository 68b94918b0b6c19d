"""Direct loads to LDS take their LDS base from m0.  The compiler uses m0 too, for register indexes known only at run time, so
a block that writes it has to say so; the register is reserved and a clobber of it is not honoured, but an output that lives
in it is.  Early, as the block reads its inputs after the write."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_02272_amd", "csrc")


def asm_blocks(text, start=r"\basm\s+volatile\s*\("):
    for m in re.finditer(start, text):
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


def instructions(block):
    return [i for i in re.split(r"\\n(?:\\t)?", "".join(re.findall(r'"([^"]*)"', re.split(r'"\s*:', block, maxsplit=1)[0] + '"'))) if i]


def test_vector_instructions_bring_their_wait_states():
    """The compiler adds wait states between vector instructions that it knows of and does not look into a block: a value just
    written may be read across lanes (two wait states before a DPP instruction, one before v_readlane), and a scalar register
    that a v_readlane just wrote by a vector instruction (two).  So a block of vector instructions begins and ends with two,
    and has two before each DPP instruction, wherever the compiler puts it.  (The one that moves a constant into a register
    needs none: the scalar unit writes its input, and what follows is ordinary arithmetic.)"""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        if not path.endswith((".hip", ".h")):
            continue
        for block in asm_blocks(open(path).read(), r"\basm(?:\s+volatile)?\s*\("):
            code = instructions(block)
            if not any(i.startswith("v_") for i in code) or code == ["v_mov_b32 %0, %1"]:
                continue
            seen += 1
            where = (os.path.basename(path), block)
            assert code[0] == "s_nop 1" and code[-1] == "s_nop 1", where
            assert all(code[n - 1] == "s_nop 1" for n, i in enumerate(code) if "_dpp" in i), where
    assert seen >= 2
