"""What the compiler gave the built library's kernels, from the metadata that it
leaves in their code object (no GPU needed)."""
import os
import struct

import pytest

from paper_2406_08186_amd import build

msgpack = pytest.importorskip("msgpack")


def _kernels():
    """The kernels' metadata: every AMDGPU ELF image in the library, its note of type 32."""
    blob, out, at = open(build.LIB, "rb").read(), [], 0
    while (at := blob.find(b"\x7fELF\x02\x01\x01\x40", at + 1)) > 0:  # 64-bit, little-endian, AMDGPU HSA
        phoff, = struct.unpack_from("<Q", blob, at + 32)
        phsize, phnum = struct.unpack_from("<HH", blob, at + 54)
        for i in range(phnum):
            kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", blob, at + phoff + i * phsize)
            if kind != 4:  # PT_NOTE
                continue
            pos, end = at + off, at + off + size
            while pos + 12 <= end:
                namesz, descsz, note = struct.unpack_from("<III", blob, pos)
                desc = pos + 12 + (namesz + 3) // 4 * 4
                if note == 32 and blob[pos + 12:pos + 18] == b"AMDGPU":
                    out += msgpack.unpackb(blob[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]
                pos = desc + (descsz + 3) // 4 * 4
    return out


@pytest.mark.skipif(not os.path.exists(build.LIB), reason="library not built")
def test_no_kernel_spills():
    """No kernel keeps registers in scratch memory: a spill is paid by every wavefront of every
    launch, most by the short ones."""
    kernels = _kernels()
    assert len(kernels) > 100 and any("k_batch_ell_lds" in k[".name"] for k in kernels)
    spilling = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels
                if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count", 0)}
    assert not spilling
