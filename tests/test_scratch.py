"""Kernels of the forward pass and of the pull by lane groups use no scratch memory (read from the built library; no GPU needed)."""
import struct

import msgpack
import pytest

from paper_2312_08656_amd import binding


def code_objects(image):
    """Notes of the AMD code objects in the library: (kernel name, scratch bytes a lane, spilled vector registers)."""
    at = image.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", image, at + 18)[0] == 224:  # EM_AMDGPU
            table, entry, n = struct.unpack_from("<Q", image, at + 40)[0], *struct.unpack_from("<HH", image, at + 58)
            for i in range(n):
                kind, _, _, offset, size = struct.unpack_from("<IQQQQ", image, at + table + i * entry + 4)
                if kind != 7:  # SHT_NOTE
                    continue
                note = at + offset
                while note < at + offset + size:
                    name, length, what = struct.unpack_from("<III", image, note)
                    body = note + 12 + (name + 3) // 4 * 4
                    if what == 32:  # NT_AMDGPU_METADATA
                        for k in msgpack.unpackb(image[body: body + length], raw=False)["amdhsa.kernels"]:
                            yield k[".name"], k[".private_segment_fixed_size"], k.get(".vgpr_spill_count", 0)
                    note = body + (length + 3) // 4 * 4
        at = image.find(b"\x7fELF", at + 4)


@pytest.mark.parametrize("kernel,least", [("spgemm_fwd_row_kernel", 100), ("spgemm_fwd_sweep_kernel", 50), ("spgemm_fwd_rmw_kernel", 10), ("pack_cbsr_kernel", 5),
                                          ("bwd_pull_lanes_kernel", 30)])
def test_no_scratch(kernel, least):
    if not binding.lib_path().exists():
        from paper_2312_08656_amd import build
        build.build()
    found = [k for k in code_objects(binding.lib_path().read_bytes()) if kernel in k[0]]
    assert len(found) >= least
    assert [k for k in found if k[1] or k[2]] == []
