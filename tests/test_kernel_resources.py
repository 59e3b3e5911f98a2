"""What the compiler gave the kernels of the built library, read from the metadata of its own code objects (no GPU): registers that
do not fit go to scratch memory, which has cost kernels four times their time without a wrong result anywhere."""
import struct

import msgpack
import pytest

from paper_2512_21450_amd import binding as B

SPILLS = {"combine16_kernelILb1E": 8}              # bytes a lane: one register, within 64 of them


def kernels(path):
    """name -> metadata of every AMDGPU kernel inside the shared object (64-bit little-endian ELF images in its bundle)."""
    blob, out, at = open(path, "rb").read(), {}, 1
    while (at := blob.find(b"\x7fELF\x02\x01", at)) > 0:
        image = blob[at:]
        at += 4
        if struct.unpack_from("<H", image, 18)[0] != 224:                      # EM_AMDGPU
            continue
        phoff, = struct.unpack_from("<Q", image, 32)
        phentsize, phnum = struct.unpack_from("<HH", image, 54)
        for i in range(phnum):
            kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", image, phoff + i * phentsize)
            end = off + size
            while kind == 4 and off + 12 <= end:                               # PT_NOTE
                name_size, desc_size, note = struct.unpack_from("<III", image, off)
                desc = off + 12 + (name_size + 3) // 4 * 4
                if note == 32 and image[off + 12:off + 12 + 6] == b"AMDGPU":   # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(image[desc:desc + desc_size], raw=False)["amdhsa.kernels"]:
                        out[k[".name"]] = k
                off = desc + (desc_size + 3) // 4 * 4
    return out


def test_no_kernel_needs_scratch_memory():
    found = kernels(B.LIB_PATH)
    for part in ("unit_kernel", "partial_kernel", "combine_kernel", "combine16_kernel", "prefill2_kernel", "prefill_kernel", "simple_kernel",
                 "token_partial_kernel", "policy_loss_kernel"):
        assert any(part in n for n in found), part
    for name, k in found.items():
        allowed = max((v for part, v in SPILLS.items() if part in name), default=0)
        assert k[".private_segment_fixed_size"] <= allowed, (name, k[".private_segment_fixed_size"], k.get(".vgpr_spill_count"))


@pytest.mark.parametrize("name,threads,lds", [("prefill2_kernelILi1ELi2E", 512, 128 * 1024), ("prefill2_kernelILi2ELi1E", 256, 64 * 1024)])
def test_two_wavefronts_a_simd(name, threads, lds):
    """The launch wants this many threads' registers (512 a lane of a SIMD) and LDS (160 KB) in a compute unit at a time."""
    k, = [k for n, k in kernels(B.LIB_PATH).items() if name in n]
    assert k[".max_flat_workgroup_size"] == threads
    assert k[".vgpr_count"] + k.get(".agpr_count", 0) <= 256 and lds * (512 // threads) + k[".group_segment_fixed_size"] * 2 <= 160 * 1024
