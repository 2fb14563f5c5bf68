"""The kernels of the built library spill no registers, but for one known form: a spilled value is reloaded inside a
streaming loop by a scratch load, and the wave then waits for every tile load in flight.  Read from
the kernel descriptors of the library's own code objects; no GPU needed."""
import struct

import pytest

import paper_2508_06526_amd as pk

# rank-16 codes at four row tiles with scores written from the loop: bytes of scratch per lane
KNOWN = {"attn_partial_gqaILi16ELi4ELi2ELb1E": 24}


def code_objects(blob):
    """The gfx950 images of every offload bundle in the file."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", blob, at + 24)
        pos = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<3Q", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + length]:
                yield blob[at + offset:at + offset + size]
            pos += 24 + length
        at += len(magic)


def scratch_bytes(image):
    """(kernel, scratch bytes per lane) from the descriptors `<kernel>.kd` of an ELF image."""
    shoff, = struct.unpack_from("<Q", image, 40)
    entry, count = struct.unpack_from("<2H", image, 58)
    # type, address, offset, size, link of every section
    sections = [(struct.unpack_from("<I", image, at + 4)[0], *struct.unpack_from("<3QI", image, at + 16))
                for at in range(shoff, shoff + entry * count, entry)]
    for kind, _, offset, size, link in sections:
        if kind != 11:                   # the dynamic symbols
            continue
        names = sections[link][2]
        for at in range(offset, offset + size, 24):
            name, _, _, where, value, _ = struct.unpack_from("<IBBHQQ", image, at)
            name = image[names + name:image.index(b"\0", names + name)].decode()
            if name.endswith(".kd"):
                _, address, start, _, _ = sections[where]
                yield name[:-3], struct.unpack_from("<I", image, start + value - address + 4)[0]


def kernels():
    if not pk.binding.is_built():
        from paper_2508_06526_amd import build
        build.build()
    with open(pk.library_path(), "rb") as f:
        return {name: size for image in code_objects(f.read()) for name, size in scratch_bytes(image)}


def spilling(found):
    allowed = lambda name: max([0] + [most for form, most in KNOWN.items() if form in name])
    return {name: size for name, size in found.items() if size > allowed(name)}


@pytest.mark.parametrize("family", ["attn_partial", "attn_combine", "attn_small", "step_", "merge_with_penalty", "utility_kernel", "route_",
                                    "evict_", "append_rows", "compress_rows", "policy_"])
def test_kernels_use_no_scratch_memory(family):
    found = {name: size for name, size in kernels().items() if family in name}
    assert found
    assert spilling(found) == {}


def test_no_kernel_of_the_library_uses_scratch_memory():
    assert spilling(kernels()) == {}
