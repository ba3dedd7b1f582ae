"""What the compiler gave the built kernels, from the metadata notes in the library's
own device code (no GPU)."""
import re
import struct

import msgpack
import pytest

from paper_1904_04884_amd import rihvr

EM_AMDGPU, PT_NOTE, NT_METADATA = 224, 4, 32


def _kernels():
    if not rihvr.LIB_PATH.exists():
        pytest.fail("librihvr.so is not built (run __graft_entry__.build())")
    data = rihvr.LIB_PATH.read_bytes()
    out = {}
    for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", data):
        o = m.start()
        if struct.unpack_from("<H", data, o + 18)[0] != EM_AMDGPU:
            continue
        phoff, = struct.unpack_from("<Q", data, o + 32)
        size, count = struct.unpack_from("<HH", data, o + 54)
        for i in range(count):
            kind, _, off, _, _, length = struct.unpack_from("<IIQQQQ", data, o + phoff + i * size)
            p = o + off
            while kind == PT_NOTE and p < o + off + length:
                name, desc, ty = struct.unpack_from("<III", data, p)
                q = p + 12 + (name + 3 & ~3)
                if ty == NT_METADATA:
                    out.update((k[".name"], k) for k in msgpack.unpackb(data[q:q + desc])["amdhsa.kernels"])
                p = q + (desc + 3 & ~3)
    return out


def test_column_transforms_keep_their_state_in_registers():
    """Their loop over planes has a tile in flight: a reload from scratch would wait for it."""
    cols = {n: k for n, k in _kernels().items() if re.search(r"k_(fwd|adj)_cols(_b)?I", n)}
    assert len(cols) == 60   # 15 lengths, single and batched
    spilled = {n: k[".private_segment_fixed_size"] for n, k in cols.items() if k[".private_segment_fixed_size"]}
    assert not spilled, spilled
