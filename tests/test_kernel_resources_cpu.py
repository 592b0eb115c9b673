"""Registers of the kernels in the built library: which of them keep values in scratch memory.

The numbers come from the metadata notes of the library's own code objects, no GPU involved."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2509_24248_amd", "libspecexit.so")

# Bytes of scratch memory per lane, at most; kernels that are not listed use none.  Each entry is stated with its timing
# beside the kernel.
SPILLS = {
    # the one-level chunk tree of the heads, for weight rows 4 KB apart
    "k_head_wide<2, 2, 2, 1, 1, 8, 4, false, 1>": 16,
    "k_head_wide<3, 2, 2, 1, 1, 8, 4, false, 1>": 20,
}


def code_objects(path):
    """The gfx950 ELF images of the library's offload bundles."""
    with open(path, "rb") as fh:
        blob = fh.read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.end()
        n, = struct.unpack_from("<Q", blob, at)
        at += 8
        if n > 16:
            continue                               # (the marker as a string, not a bundle)
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name and size:
                yield blob[m.start() + off:m.start() + off + size]


def kernels(elf):
    """Metadata of the kernels of one code object: the msgpack map of its AMDGPU note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        if kind != 7:                              # SHT_NOTE
            continue
        at = off
        while at < off + size:
            namesz, descsz, typ = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if typ == 32:                          # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[desc:desc + descsz]).get("amdhsa.kernels", [])
            at = desc + (descsz + 3) // 4 * 4


def readable(mangled):
    """Name and integral template arguments of a mangled kernel: enough to tell the instantiations apart."""
    m = re.match(r"_ZN2sx12_GLOBAL__N_1(\d+)", mangled)
    if not m:
        return mangled
    end = m.end() + int(m.group(1))
    args = re.match(r"I((?:L[ib]\d+E|[tf])+)E", mangled[end:])
    if not args:
        return mangled[m.end():end]
    names = [{"t": "unsigned short", "f": "float"}.get(a) or (a[2:-1] if a[1] == "i" else ("true" if a[2] == "1" else "false"))
             for a in re.findall(r"L[ib]\d+E|[tf]", args.group(1))]
    return f"{mangled[m.end():end]}<{', '.join(names)}>"


@pytest.mark.skipif(not os.path.exists(LIB), reason="libspecexit.so not built")
def test_heads_of_other_depths_have_a_form_that_does_not_spill():
    # the same wave splits without the tree (last argument 0) exist beside the ones listed above
    names = {readable(k[".name"]) for elf in code_objects(LIB) for k in kernels(elf)}
    for n in SPILLS:
        if n.startswith("k_head_wide<") and not n.startswith("k_head_wide<3, 2, 2, 1,"):      # (there the other form shares a tile)
            assert n.replace("false, 1>", "false, 0>") in names


@pytest.mark.skipif(not os.path.exists(LIB), reason="libspecexit.so not built")
def test_no_kernel_spills_unless_it_is_listed():
    found = {}
    for elf in code_objects(LIB):
        for k in kernels(elf):
            found[readable(k[".name"])] = k[".private_segment_fixed_size"]
    assert len(found) > 50 and any(n.startswith("k_attn_ring<") for n in found)
    over = {n: b for n, b in found.items() if b > SPILLS.get(n, 0)}
    assert not over, f"kernels with more scratch memory than stated: {over}"

