"""Layout of the built kernels, from the metadata the compiler writes beside them
(no GPU needed)."""
import os
import struct

import msgpack

import paper_2405_12497_amd

LIB = os.path.join(os.path.dirname(paper_2405_12497_amd.__file__), "librabitq.so")


def _code_objects():
    blob, at = open(LIB, "rb").read(), 0
    while (at := blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        count, o = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, o)
            if b"gfx950" in blob[o + 24:o + 24 + n]:
                yield blob[at + off:at + off + size]
            o += 24 + n
        at += 24


def _kernels():
    out = {}
    for elf in _code_objects():
        at = elf.index(b"AMDGPU\0")   # the name of the metadata's ELF note
        size = struct.unpack_from("<I", elf, at - 8)[0]
        meta = msgpack.unpackb(elf[at + 8:at + 8 + size], raw=False, strict_map_key=False)
        out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
    return out


def test_block_rerank_reads_its_query_aligned():
    """The block rerank's dynamic LDS begins after the static part and holds the query,
    which is read as float4 at a multiple of 16 bytes from there."""
    forms = {n: k for n, k in _kernels().items() if "k_finalizeILb" in n}
    assert len(forms) == 4
    for name, k in forms.items():
        assert k[".group_segment_fixed_size"] % 16 == 0, name
