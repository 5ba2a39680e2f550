"""What the compiler gave the kernels of the built library, read from the
metadata of its gfx950 code objects (no GPU needed).

Registers that do not fit are kept in scratch memory.  The compiler waits for
such a reload as for any load, and memory operations complete in order, so a
reload inside a loop also waits for the direct loads to LDS that the kernel
has in flight on purpose: a kernel with scratch has lost its pipeline.
"""
import struct

import msgpack

from paper_2607_06827_amd import speechkv as skv

ELF_MACHINE_AMDGPU = 224
NOTE_METADATA = 32  # NT_AMDGPU_METADATA: MessagePack


def _notes(elf):
    """(type, description) of the notes of a 64-bit little-endian ELF image."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        at, end = offset, offset + size
        while kind == 4 and at + 12 <= end:  # PT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3 & ~3)
            yield note, elf[at:at + desc]
            at += desc + 3 & ~3


def kernels():
    """Metadata of every kernel of the library by (mangled) name."""
    image = open(skv.LIBRARY_PATH, "rb").read()
    found, at = {}, image.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", image, at + 18)[0] == ELF_MACHINE_AMDGPU:
            for note, desc in _notes(image[at:]):
                if note == NOTE_METADATA:
                    for k in msgpack.unpackb(desc)["amdhsa.kernels"]:
                        found[k[".name"]] = k
        at = image.find(b"\x7fELF", at + 4)
    return found


def test_the_library_holds_its_kernels():
    names = " ".join(kernels())
    for k in ("pool_kv_kernel", "decode_kernel", "prefill_kernel_lds", "prefill_kernel_fused", "prefill_f32_kernel",
              "prefill_bwd_dq16_kernel", "prefill_bwd_dkdv16_kernel", "prefill_bwd_dkdv_f32_kernel",
              "pool_bwd_kernel", "pool_hidden_kernel"):
        assert k in names, k


def test_no_kernel_uses_scratch():
    assert not {n: k[".private_segment_fixed_size"] for n, k in kernels().items()
                if k[".private_segment_fixed_size"] or k[".uses_dynamic_stack"]}
