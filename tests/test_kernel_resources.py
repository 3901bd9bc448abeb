"""What the compiler made of the kernels, from the metadata of the code objects in the built library (no GPU needed)."""
import struct

import msgpack

from gpu_util import ensure_built
from paper_2505_11170_amd import binding

AMDGPU = 224   # e_machine


def kernels():
    """The amdhsa metadata of every kernel in libgws.so, by name."""
    ensure_built()
    with open(binding.library_path(), "rb") as f:
        data = f.read()
    out, at = {}, data.find(b"\x7fELF", 1)
    while at >= 0:
        machine, = struct.unpack_from("<H", data, at + 18)
        if machine == AMDGPU:
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phentsize, phnum = struct.unpack_from("<HH", data, at + 54)
            for i in range(phnum):
                kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + i * phentsize)
                p, end = at + offset, at + offset + size
                while kind == 4 and p + 12 <= end:   # PT_NOTE: name size, contents' size, type, each padded to four bytes
                    name, desc, note = struct.unpack_from("<III", data, p)
                    p += 12 + (name + 3) // 4 * 4
                    if note == 32:                   # NT_AMDGPU_METADATA
                        out.update((k[".name"], k) for k in msgpack.unpackb(data[p:p + desc])["amdhsa.kernels"])
                    p += (desc + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 1)
    return out


def test_kernels_use_no_scratch():
    # a kernel with scratch starts up to half a microsecond later: the products and what rides in them, the gradients, the sampling passes
    found = kernels()
    assert len(found) > 100
    for part in ("gemm256", "gemm128", "gemm_stream_kernel", "gemm_stream_tn", "gemm_rows", "sample_fwd", "sample_bwd"):
        mine = [k for k in found.values() if part in k[".name"]]
        assert mine and not [k[".name"] for k in mine if k[".private_segment_fixed_size"] != 0]
