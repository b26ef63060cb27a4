"""Registers, LDS and scratch of the built kernels, read from the code objects' metadata in libspts.so (no GPU needed)."""
import os
import re
import struct

import msgpack
import pytest

from paper_2601_13155_amd import binding

CSRC = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")


@pytest.fixture(scope="module")
def kernels():
    """{mangled name: metadata map} of every gfx950 kernel in the library."""
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    data = open(binding.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        base, at = m.start(), m.start() + 32
        for _ in range(struct.unpack_from("<Q", data, base + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + n]
            at += 24 + n
            if size and b"gfx950" in target:
                out.update(_notes(data[base + off:base + off + size]))
    assert out, "no gfx950 code object in the library"
    return out


def _notes(elf):
    """The AMDGPU metadata note (MessagePack) of one code object: {kernel name: map}."""
    sections = struct.unpack_from("<Q", elf, 0x28)[0]
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind = struct.unpack_from("<I", elf, sections + i * entry + 4)[0]
        at = struct.unpack_from("<Q", elf, sections + i * entry + 24)[0]
        if kind == 7:   # SHT_NOTE
            name_size, size, _ = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name_size + 3) // 4 * 4
            meta = msgpack.unpackb(elf[body:body + size], raw=False)
            return {k[".name"]: k for k in meta["amdhsa.kernels"]}
    return {}


def _named(kernels, part):
    found = {n: k for n, k in kernels.items() if part in n}
    assert found, f"no kernel named {part}"
    return found


def test_long_row_topk_leaves_room_for_two_workgroups(kernels):
    """512 long rows are two workgroups per CU: each within half of its 160 KB of LDS and of its registers (8 wavefronts per SIMD)."""
    src = open(os.path.join(CSRC, "kernels_topk.hip")).read()
    dynamic = int(re.search(r"constexpr int T13_LDS_BYTES = (\d+) \* 1024;", src).group(1)) * 1024
    for part in ("topk_long_kernel", "topk_once_kernel"):
        for name, k in _named(kernels, part).items():
            assert k[".group_segment_fixed_size"] + dynamic <= 80 * 1024, name
            assert k[".vgpr_count"] <= 64 and k[".private_segment_fixed_size"] == 0, name


def test_fp32_attention_scratch(kernels):
    """Head dimensions above 128 exceed a lane's 512 registers by the row pieces of a query and a key block; no more of the loop than that goes to
    scratch memory (with 1448 bytes a lane the attention of 6000 rows takes 1.9 times as long as with 1300)."""
    for name, k in _named(kernels, "attention_f32_kernel").items():
        d = int(re.search(r"Li(\d+)E", name).group(1))
        assert k[".private_segment_fixed_size"] <= {32: 0, 64: 16, 128: 0, 256: 1320}[d], name
