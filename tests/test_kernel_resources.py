"""Scratch memory of the kernels in the built library, from its code objects.

A queue holds scratch for every wavefront the device can run (256 compute
units of 32), whatever a launch needs: 128 bytes per lane are 64 MiB per
queue, and the local kernels run on several queues at once."""
import struct

import msgpack

from paper_2410_24138_amd import nls

EM_AMDGPU, SHT_NOTE, NT_METADATA = 224, 7, 32
LIMIT = 128


def kernels(path):
    """Metadata of every kernel in the device code objects embedded in path."""
    data = open(path, "rb").read()
    out, at = {}, data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff = struct.unpack_from("<Q", data, at + 40)[0]
            size, num = struct.unpack_from("<HH", data, at + 58)
            for s in range(num):
                kind, off, length = struct.unpack_from("<4xI16xQQ", data, at + shoff + s * size)
                if kind != SHT_NOTE:
                    continue
                p, end = at + off, at + off + length
                while p < end:
                    nn, nd, nt = struct.unpack_from("<III", data, p)
                    d = p + 12 + (nn + 3) // 4 * 4
                    if nt == NT_METADATA:
                        for k in msgpack.unpackb(data[d:d + nd])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    p = d + (nd + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


def test_scratch_of_every_kernel():
    ks = kernels(nls.LIB_PATH)
    assert any("k_local_newton" in n for n in ks) and any("k_gemm_bf16" in n for n in ks)
    over = {n: k[".private_segment_fixed_size"] for n, k in ks.items()
            if k[".private_segment_fixed_size"] > LIMIT}
    assert not over
