"""CPU check of the buffer accesses in the kernel sources.  The range check of a raw buffer access covers the vector
offset; the compiler's contract leaves the scalar offset out of it.  A request that is meant to be out of range (it
then reads zero and moves nothing) must therefore carry the out-of-range value in its vector offset: through the
scalar offset it could read two gigabytes past the buffer, and no comparison of results would show it."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_17870_amd", "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")))
OUT_OF_RANGE = {"NOWHERE", "OOR", "ST_OOR"}
# position of the scalar offset among the arguments
CALLS = [(re.compile(r"__builtin_amdgcn_raw_buffer_(?:load|store)_\w+\s*\("), -2),
         (re.compile(r"__builtin_amdgcn_raw_ptr_buffer_load_lds\s*\("), 4),
         (re.compile(r"\bgb_fetch\s*\("), -1)]


def code_of(path):
    text = open(path).read()
    text = re.sub(r"/\*.*?\*/", lambda m: " " * len(m.group()), text, flags=re.S)
    return re.sub(r"//[^\n]*", lambda m: " " * len(m.group()), text)


def arguments(code, start):
    """The arguments of a call whose opening parenthesis ends at `start`."""
    depth, out, at = 1, [], start
    for i in range(start, len(code)):
        c = code[i]
        if c in "([{":
            depth += 1
        elif c in ")]}":
            depth -= 1
            if depth == 0:
                return out + [code[at:i]]
        elif c == "," and depth == 1:
            out.append(code[at:i])
            at = i + 1
    raise AssertionError("call without an end")


def reaches_out_of_range(expr, code, before, seen=()):
    """Whether the expression, its variables replaced by their latest definitions, can be an out-of-range value."""
    if re.search(r"0x7fff[0-9a-f]{4}", expr):
        return True
    for name in set(re.findall(r"[A-Za-z_]\w*", expr)) - set(seen):
        if name in OUT_OF_RANGE:
            return True
        defs = [m for m in re.finditer(r"\b" + name + r"\s*=(?!=)\s*([^;]*);", code[:before])]
        if defs and reaches_out_of_range(defs[-1].group(1), code, defs[-1].start(), (*seen, name)):
            return True
    return False


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_no_out_of_range_value_in_a_scalar_offset(path):
    code = code_of(path)
    for pattern, position in CALLS:
        for m in pattern.finditer(code):
            soff = arguments(code, m.end())[position].strip()
            line = code.count("\n", 0, m.start()) + 1
            assert not reaches_out_of_range(soff, code, m.start()), f"{os.path.basename(path)}:{line}: scalar offset '{soff}'"


def test_the_check_finds_one():
    code = "const int hoff = kb < KB ? kb * 256 : NOWHERE;\n f(__builtin_amdgcn_raw_buffer_load_b32(rs, v, hoff, 0));"
    m = CALLS[0][0].search(code)
    assert reaches_out_of_range(arguments(code, m.end())[-2], code, m.start())
    assert not reaches_out_of_range("kb * 256", code, m.start())
