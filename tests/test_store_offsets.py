"""Wide buffer stores of the built library (its own gfx950 code, no GPU).

A buffer store of 12 or 16 bytes with a register as scalar offset gets no wait
state before the next instruction, which may then overwrite the data registers
while the store still reads them.  Every such store has to carry its offset in
the lane offset, with the constant 0 as scalar offset.
"""
import os
import re
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2105_06806_amd", "libedx.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of the library's offload bundles."""
    for m in re.finditer(MAGIC, data):
        base = m.start()
        count, = struct.unpack_from("<Q", data, base + len(MAGIC))
        pos = base + len(MAGIC) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24: pos + 24 + tlen]
            pos += 24 + tlen
            if size and target.endswith(b"gfx950"):
                yield data[base + off: base + off + size]


@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(OBJDUMP)),
                    reason="libedx.so or llvm-objdump not there")
def test_wide_stores_have_no_scalar_offset(tmp_path):
    paths = []
    for k, blob in enumerate(code_objects(open(LIB, "rb").read())):
        paths.append(tmp_path / f"{k}.co")
        paths[-1].write_bytes(blob)
    assert paths

    def stores(path):
        txt = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True,
                             check=True).stdout
        return re.findall(r"buffer_store_dwordx[34] .*", txt)

    with ThreadPoolExecutor(4) as ex:
        found = [s for r in ex.map(stores, paths) for s in r]
    assert found        # both passes with wide stores are there
    # operands: data, lane offset, resource, scalar offset
    bad = [s for s in found if re.split(r",\s*", s)[3].split()[0] != "0"]
    assert not bad, bad[:5]
