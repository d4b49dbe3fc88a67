"""The built library's kernels and scratch memory, read from its kernel descriptors (no GPU): the kernels of the usual calls are held to
register limits that their occupancy needs, and have to fit them without spilling."""
import os
import struct

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_05688_amd", "libvatt.so")
EM_AMDGPU, SHT_SYMTAB, SHT_DYNSYM = 224, 2, 11

# the selection kernel with rare options, which is over its limit by two registers
MAY_SPILL = ("head_kernelILi512ELi0ELb0ELb0ELi0ELb1E",)


def _scratch_bytes(path):
    """{kernel: bytes of scratch memory per thread}: the second word of every kernel's descriptor in the embedded gfx950 objects."""
    data = open(path, "rb").read()
    out, at = {}, data.find(b"\x7fELF\x02\x01")
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, count = struct.unpack_from("<HH", data, at + 58)
            sections = [struct.unpack_from("<IIQQQQIIQQ", data, at + shoff + i * size) for i in range(count)]
            for _, kind, _, _, off, length, link, _, _, entry in sections:
                if kind not in (SHT_SYMTAB, SHT_DYNSYM):
                    continue
                for s in range(off, off + length, entry):
                    name, _, _, section, value, _ = struct.unpack_from("<IBBHQQ", data, at + s)
                    start = at + sections[link][4] + name
                    text = data[start:data.index(b"\0", start)].decode()
                    if text.endswith(".kd"):
                        home = sections[section]
                        out[text[:-3]] = struct.unpack_from("<I", data, at + home[4] + value - home[3] + 4)[0]
        at = data.find(b"\x7fELF\x02\x01", at + 4)
    return out


def test_kernels_keep_out_of_scratch_memory():
    scratch = _scratch_bytes(LIB)
    assert sum("head_kernel" in k for k in scratch) >= 20, sorted(scratch)
    spilled = {k: b for k, b in scratch.items() if b and not any(m in k for m in MAY_SPILL)}
    assert not spilled, spilled
