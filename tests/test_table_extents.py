"""Extents of the sector tables that a product reads in words (no GPU).

The product on 16-byte lanes reads the impurity patterns of two rows as one
16-bit word through a buffer resource.  The bytes that the resource covers, the
bytes that the table builder allocates and clears and the bytes that the
memory estimate of a sector counts are one expression, which covers the last
word of an odd table.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_06806_amd", "csrc")


def _src(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def test_pattern_table_is_allocated_as_it_is_read():
    hv, tables = _src("hv.hip"), _src("tables.hip")
    # (the row-a-lane passes before and after it read single bytes)
    lanes = hv[hv.index("void k_hv_vec("):hv.index("// ---------------------------------------------------------------- fused launches")]
    reads = re.findall(r"make_buffer_rsrc\(\s*const_cast<uint8_t\*>\(a\.pup\), 0, \(int\)([^,]+), ", lanes)
    assert reads == ["pat_bytes(dup)"]
    assert re.findall(r"dalloc\(S, &T\.pat, (.+)\)\);", tables) == ["pat_bytes(D)"]
    assert "pat_bytes(D) > D) pat[D] = 0;" in tables
    assert "(size_t)pat_bytes(D)" in tables[tables.index("size_t sector_table_bytes"):]


@pytest.mark.parametrize("rows", [1, 2, 3, 252, 461, 462, 3003, 12869, 12870])
def test_pattern_table_covers_the_last_word(rows):
    expr = re.search(r"int64_t pat_bytes\(int64_t D\) \{ return (.+); \}", _src("edx_internal.h")).group(1)
    size = eval(expr.replace("/", "//"), {"D": rows})
    # the word of the last pair of rows ends at the next even byte
    assert rows <= size <= rows + 1 and size >= (rows - 1) // 2 * 2 + 2
