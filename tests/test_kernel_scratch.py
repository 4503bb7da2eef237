"""The FP32 field kernels of the integrators reserve no scratch memory: a
kernel with a scratch reservation makes the runtime allocate device memory at
its first launch on a queue, inside an integrator call.  Read from the metadata
of the built library's gfx950 code object."""
import os
import struct

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2608_15253_amd", "libmmx.so")


def _code_object(blob):
    """The gfx950 entry of the library's offload bundle."""
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    assert at >= 0, "no uncompressed offload bundle"
    n, = struct.unpack_from("<Q", blob, at + 24)
    p = at + 32
    for _ in range(n):
        off, size, idlen = struct.unpack_from("<QQQ", blob, p)
        name = blob[p + 24:p + 24 + idlen]
        p += 24 + idlen
        if b"gfx950" in name:
            return blob[at + off:at + off + size]
    raise AssertionError("no gfx950 code object")


def _kernels(elf):
    """{kernel name: scratch bytes} of the AMDGPU metadata note."""
    import msgpack
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        ptype, _, off, _, _, filesz = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        if ptype != 4:  # PT_NOTE
            continue
        p, end = off, off + filesz
        while p < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + namesz].rstrip(b"\0")
            d = p + 12 + (namesz + 3) // 4 * 4
            if name == b"AMDGPU" and ntype == 32:
                meta = msgpack.unpackb(elf[d:d + descsz])
                return {k[".name"]: k[".private_segment_fixed_size"]
                        for k in meta["amdhsa.kernels"]}
            p = d + (descsz + 3) // 4 * 4
    raise AssertionError("no AMDGPU metadata")


def test_fp32_field_kernels_reserve_no_scratch():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with open(LIB, "rb") as f:
        kernels = _kernels(_code_object(f.read()))
    fields = {k: v for k, v in kernels.items() if "k_fieldsIf" in k}
    assert len(fields) >= 7  # every mode
    assert {k: v for k, v in fields.items() if v} == {}
