"""Loads in inline assembly.  The compiler takes the output registers of an asm block as written when the block ends and may read, move or reuse
them at once, so a block that loads into registers waits for the load itself; loads that are waited for later are ordinary loads or builtins,
which the compiler counts.  (Copies into LDS have no output registers and may be waited for anywhere.)"""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2102_10485_amd", "csrc")
LOAD = re.compile(r"\b(ds_read|ds_load|buffer_load|global_load|flat_load|scratch_load|s_load|s_buffer_load)")


def asm_blocks(text):
    for m in re.finditer(r"\basm\s+(?:volatile\s*)?\(", text):
        depth, i = 1, m.end()
        quoted = False
        while depth:
            ch = text[i]
            if ch == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(ch, 0)
            i += 1
        yield text[m.end():i - 1]


def loads_without_a_wait(text):
    return [b for b in asm_blocks(text) if LOAD.search(b) and re.search(r'"[=+]&?[vas]"', b) and "s_waitcnt" not in b]


def test_the_search_finds_such_a_block():
    bad = 'asm volatile("ds_read_b128 %0, %1" : "=v"(d) : "v"(addr) : "memory");'
    assert loads_without_a_wait(bad) and not loads_without_a_wait(bad.replace('%1"', '%1\\n\\ts_waitcnt lgkmcnt(0)"'))


def test_every_load_is_waited_for_where_it_is_written():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        assert loads_without_a_wait(open(path).read()) == [], path
