"""The built library's kernels keep their values in registers: none has scratch
memory (spilled registers, or arrays indexed at run time), which the decode
path's speed rests on.  Read from the metadata note of the library's own code
objects."""
import struct

import pytest

from paper_2609_38169_amd import stepq

EM_AMDGPU = 224
NT_AMDGPU_METADATA = 32


def _notes(elf):
    """(owner, type, payload) of an ELF image's note sections."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + i * size + 0x18)
        if kind != 7:
            continue
        end = off + length
        while off + 12 <= end:
            n, d, t = struct.unpack_from("<III", elf, off)
            name = off + 12
            data = name + (n + 3) // 4 * 4
            yield elf[name:name + n].rstrip(b"\0"), t, elf[data:data + d]
            off = data + (d + 3) // 4 * 4


def _kernels():
    msgpack = pytest.importorskip("msgpack")
    image = open(stepq.LIB_PATH, "rb").read()
    at, out = image.find(b"\x7fELF", 1), []
    while at >= 0:
        if struct.unpack_from("<H", image, at + 18)[0] == EM_AMDGPU:
            for owner, kind, data in _notes(image[at:]):
                if owner == b"AMDGPU" and kind == NT_AMDGPU_METADATA:
                    out += msgpack.unpackb(data, raw=False)["amdhsa.kernels"]
        at = image.find(b"\x7fELF", at + 4)
    return out


def test_no_kernel_uses_scratch():
    stepq.lib()
    kernels = _kernels()
    names = [k[".name"] for k in kernels]
    for part in ("decode_kernel", "refit_kernel", "rowmax_kernel", "load_kernel", "dequant_kernel"):
        assert any(part in n for n in names), part
    bad = {k[".name"]: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"])
           for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not bad, bad


def test_frozen_bodies_keep_eight_waves():
    """The frozen steps' bodies for fp32 activations at d_v = 128, but for the
    one of any mix (layout 0), fit 64 registers: 8 waves per SIMD, on which a
    launch's rounds rest."""
    stepq.lib()
    wide = {k[".name"]: k[".vgpr_count"] for k in _kernels()
            if "decode_kernelILi128ELb0E" in k[".name"] and "ELi0ELb" not in k[".name"] and k[".vgpr_count"] > 64}
    assert not wide, wide
