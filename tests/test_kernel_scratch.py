"""No kernel of the built library keeps registers or arrays in scratch memory (a
private segment costs its stores and loads on every lane): read from the kernel
descriptors (`<kernel>.kd`, whose bytes 4-7 hold the private segment's size) of the
gfx950 images inside libdg.so."""
import struct
from pathlib import Path

import paper_2008_09441_amd

EM_AMDGPU, SHT_DYNSYM = 224, 11


def _private_segments(data):
    sizes, at = {}, data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, n, _ = struct.unpack_from("<HHH", data, at + 58)
            # per section: name, type, flags, address, offset, size, link, info, align, entry
            secs = [struct.unpack_from("<IIQQQQIIQQ", data, at + shoff + i * size) for i in range(n)]
            for s in (s for s in secs if s[1] == SHT_DYNSYM):
                names = at + secs[s[6]][4]
                for sym in range(at + s[4], at + s[4] + s[5], s[9]):
                    name, _, _, shndx, value, _ = struct.unpack_from("<IBBHQQ", data, sym)
                    name = data[names + name:data.index(b"\0", names + name)].decode()
                    if name.endswith(".kd"):
                        home = secs[shndx]
                        kd = at + home[4] + value - home[3]
                        sizes[name] = struct.unpack_from("<I", data, kd + 4)[0]
        at = data.find(b"\x7fELF", at + 1)
    return sizes


def test_no_kernel_uses_scratch():
    lib = Path(paper_2008_09441_amd.__file__).parent / "libdg.so"
    sizes = _private_segments(lib.read_bytes())
    assert any("stage_bt_batch" in k for k in sizes) and any("stage_bx" in k for k in sizes)
    assert not {k: v for k, v in sizes.items() if v}
