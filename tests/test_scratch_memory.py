"""What the compiler gave the kernels of the built library: none keeps its accumulators in scratch memory (a lambda that it stops inlining
puts them there, and the kernel still gives the right results, thirty times slower)."""
import struct

import msgpack

from paper_1909_09577_amd import binding as nm

NOTE_METADATA = 32  # NT_AMDGPU_METADATA


def _metadata(elf):
    """The metadata note of a 64-bit little-endian code object that starts at elf[0]."""
    at, = struct.unpack_from("<Q", elf, 0x20)
    size, count = struct.unpack_from("<HH", elf, 0x36)
    for i in range(count):
        kind, _, offset, _, _, length = struct.unpack_from("<IIQQQQ", elf, at + i * size)
        end = offset + length
        while kind == 4 and offset < end:  # PT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, offset)
            body = offset + 12 + (name + 3) // 4 * 4
            if note == NOTE_METADATA:
                return msgpack.unpackb(elf[body:body + desc])
            offset = body + (desc + 3) // 4 * 4


def _kernels():
    nm.lib()
    lib = open(nm.LIB_PATH, "rb").read()
    at = lib.find(b"\x7fELF", 1)
    while at >= 0:
        yield from (_metadata(lib[at:]) or {}).get("amdhsa.kernels", [])
        at = lib.find(b"\x7fELF", at + 1)


def test_no_kernel_works_in_scratch_memory():
    """A few spilled registers are at most 128 bytes a lane; the smallest accumulator tile is 256."""
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for k in _kernels()}
    assert len(scratch) > 200 and any("pointwise_gemm_kernelILb1ELi4ELi4" in n for n in scratch)
    assert not {n: s for n, s in scratch.items() if s > 128}
