"""What the compiler made of the kernels, from the metadata of the built library's own code objects (host only)."""
import re
import struct

import pytest

from paper_2210_06223_amd import build


def _kernels(path):
    """[(name, metadata)] of every gfx950 kernel in the library."""
    msgpack = pytest.importorskip("msgpack")
    data = open(path, "rb").read()
    out = []
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start() + 24
        n, at = struct.unpack_from("<Q", data, at)[0], at + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" not in target or not size:
                continue
            elf = data[m.start() + off:m.start() + off + size]
            shoff, = struct.unpack_from("<Q", elf, 0x28)
            entsize, count = struct.unpack_from("<HH", elf, 0x3A)
            for i in range(count):
                kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
                start, length = struct.unpack_from("<QQ", elf, shoff + i * entsize + 0x18)
                if kind != 7:                                          # SHT_NOTE
                    continue
                namesz, descsz, _ = struct.unpack_from("<III", elf, start)
                desc = start + 12 + (namesz + 3) // 4 * 4
                meta = msgpack.unpackb(elf[desc:desc + descsz])
                out += [(k[".name"], k) for k in meta.get("amdhsa.kernels", [])]
    return out


@pytest.mark.parametrize("path", [build.LIB, build.LIB_CHECK], ids=["library", "check build"])
def test_no_kernel_keeps_registers_or_arrays_in_scratch_memory(path):
    """A k-loop that the compiler does not unroll in full decides its counted barriers at run time and keeps its rings where the
    loop counter can index them; a reload from scratch memory in it waits for every weight requested before."""
    kernels = _kernels(path)
    names = " ".join(n for n, _ in kernels)
    for k in ("fused_bneck", "stream_bneck", "tiled_conv", "slab_conv", "rows_conv", "masker", "bneck_generic"):
        assert k in names, k
    bad = [(n, k[".private_segment_fixed_size"], k.get(".vgpr_spill_count")) for n, k in kernels
           if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")]
    assert not bad, bad
