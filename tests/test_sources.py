"""Rules that the kernel sources keep, checked on their text (CPU)."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = sorted(glob.glob(os.path.join(ROOT, "paper_2607_10661_amd", "csrc", "*.h*")))


def asm_statements(text):
    """The argument text of every asm statement (parentheses matched)."""
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text[m.end():i - 1]


def test_no_register_load_without_its_wait():
    # an inline-asm load into a VGPR is taken as complete by the compiler, which may
    # copy or reuse the register while the data is on its way: such a load has its
    # wait in the same statement, or is an ordinary load
    load = re.compile(r"\b(global|flat|buffer|scratch)_load_(?!lds)|\bds_read|\bs_load|\bs_buffer_load")
    found, seen = [], 0
    for path in SOURCES:
        for body in asm_statements(open(path).read()):
            seen += 1
            if load.search(body) and re.search(r'"=&?[vsa]"', body) and "global_load_lds" not in body \
                    and "s_waitcnt" not in body:
                found.append((os.path.basename(path), body.strip()[:60]))
    assert len(SOURCES) >= 8 and seen >= 8
    assert not found
