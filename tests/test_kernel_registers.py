"""What the built kernels occupy, from the metadata of the code object in the library."""
import os
import re
import struct

import msgpack
import pytest

import paper_2502_14866_amd as L


def _kernels(path):
    """Metadata of every kernel in the AMDGPU code objects of a shared library, by mangled name."""
    data, out, at = open(path, "rb").read(), {}, 0
    while (at := data.find(b"\x7fELF", at + 1)) > 0:
        if struct.unpack_from("<H", data, at + 18)[0] != 224:  # EM_AMDGPU
            continue
        table, entry, count = struct.unpack_from("<Q", data, at + 40)[0], *struct.unpack_from("<HH", data, at + 58)
        for i in range(count):
            kind, _, _, offset, size = struct.unpack_from("<IQQQQ", data, at + table + i * entry + 4)
            if kind != 7:  # SHT_NOTE
                continue
            name_size, body_size, note = struct.unpack_from("<III", data, at + offset)
            if note != 32:  # NT_AMDGPU_METADATA
                continue
            body = at + offset + 12 + (name_size + 3) // 4 * 4
            for kernel in msgpack.unpackb(data[body:body + body_size], strict_map_key=False)["amdhsa.kernels"]:
                out[kernel[".name"]] = kernel
    return out


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(L.library_path()):
        from paper_2502_14866_amd.build import build_library

        build_library()
    return _kernels(L.library_path())


def test_decode_kernels_leave_room_for_two_workgroups(kernels):
    """Four wavefronts each, one to a SIMD: 256 of its 512 registers a workgroup, half of the 160 KiB of shared memory.
    Pages of 128 tokens under six and more heads need more registers and run alone."""
    seen = 0
    for name, k in kernels.items():
        m = re.search(r"sparse_decode_kernelINS_\d+B?F16ELi(\d+)ELi(\d+)ELi(\d+)E", name)
        if not m:
            continue
        heads, page, _ = map(int, m.groups())
        seen += 1
        assert k[".private_segment_fixed_size"] == 0, name
        if page == 128 and heads > 5:
            continue
        assert k[".vgpr_count"] <= 256 and k[".group_segment_fixed_size"] <= 80 * 1024, name
    assert seen == 2 * 8 * 6  # types, heads per group, (page, bits)


def test_prefill_kernels_use_no_scratch(kernels):
    found = [k for name, k in kernels.items() if "sparse_prefill_kernel" in name]
    assert len(found) == 2 * (3 + 2 + 3 + 2 + 2)  # types, slices over prompts, listed masks, pages of 16, 8 and 4 bits
    assert all(k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 256 for k in found)


def test_half_prefill_workgroups_go_two_to_a_compute_unit(kernels):
    """Four wavefronts each, one to a SIMD, and no scratch; chunks in pieces: no scratch either."""
    halves = [k for name, k in kernels.items() if "prefill_half_kernel" in name or "prefill_hasty_kernel" in name]
    assert len(halves) == 2 * (3 + 1)  # types, (prompts, listed masks, pages) and prompts whose longest walk goes first
    assert all(k[".vgpr_count"] <= 256 and k[".group_segment_fixed_size"] <= 80 * 1024 for k in halves)
    pieces = [k for name, k in kernels.items() if "pieces_kernel" in name]
    assert len(pieces) == 2 * (3 + 1)  # types, widths of the pages and the kernel that puts pieces together
    assert all(k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 256 for k in halves + pieces)


def test_fold_and_streams_use_no_scratch(kernels):
    """The body of a whole walk in slices and that which puts pieces together, in one kernel of eight wavefronts."""
    both = [k for name, k in kernels.items() if "fold_and_streams_kernel" in name]
    assert len(both) == 2 * (2 + 1 + 1)  # types, 16-bit pages in two and four slices, 8- and 4-bit pages in two
    assert all(k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 256 for k in both)
    assert all(k[".group_segment_fixed_size"] <= 160 * 1024 for k in both)


def test_selector_runs_of_one_launch_use_no_scratch(kernels):
    """Five workgroups of four wavefronts to a compute unit at most: 102 registers each."""
    found = [k for name, k in kernels.items() if "select_all_kernel" in name]
    assert len(found) == 2
    assert all(k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 102 for k in found)
