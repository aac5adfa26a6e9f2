"""Scratch memory of the built kernels, from the code objects in the library:
none spills to it beyond the few listed bytes."""
import os
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_00477_amd", "libstencil_mi355.so")

# mangled-name parts of the kernels that use a few bytes of scratch per lane
# (measured faster with them than with a wave less), and how many
FEW = {"valu3d_kernel": 16, "valu3d_batch_kernel": 16,
       "valu3d_box_kernel": 12,      # float32 r = 2, held to six waves per SIMD
       "fused3d_batch_kernel": 8}    # float32 Star-3D3R T = 2


def _code_objects(data):
    """The gfx950 code objects of the offload bundles in the library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


def _kernels(obj):
    """Kernel entries of a code object's metadata note."""
    import msgpack
    (shoff,) = struct.unpack_from("<Q", obj, 0x28)
    entsize, num = struct.unpack_from("<HH", obj, 0x3A)
    for k in range(num):
        typ, = struct.unpack_from("<I", obj, shoff + k * entsize + 4)
        if typ != 7:  # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", obj, shoff + k * entsize + 0x18)
        pos, end = off, off + size
        while pos < end:
            nlen, dlen, kind = struct.unpack_from("<III", obj, pos)
            body = pos + 12 + (nlen + 3) // 4 * 4
            if kind == 32:  # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(obj[body:body + dlen])["amdhsa.kernels"]
            pos = body + (dlen + 3) // 4 * 4


def test_no_kernel_spills_to_scratch():
    pytest.importorskip("msgpack")
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with open(LIB, "rb") as f:
        data = f.read()
    total, bad = 0, []
    for obj in _code_objects(data):
        for k in _kernels(obj):
            total += 1
            allowed = max((b for part, b in FEW.items() if part in k[".name"]), default=0)
            if k[".private_segment_fixed_size"] > allowed:
                bad.append((k[".name"], k[".private_segment_fixed_size"]))
    assert total > 500
    assert not bad, bad[:5]


def test_compensated_passes_have_matrix_kernels():
    """The vector kernels of the compensated mode only redo bands: every plan of
    it that can be made has a matrix kernel at each depth its runs may use, and
    no three-dimensional plan of it exists."""
    import paper_2603_00477_amd as stl
    made = 0
    for shape in ("star", "box"):
        for d in (2, 3):
            for r in (1, 2, 3, 4, 7):
                K = (2 * r + 1) ** d if shape == "box" else 2 * d * r + 1
                for T in range(1, 9):
                    try:
                        stl.Plan(shape, d, r, [1.0 / K] * K, (64,) * d, T=T, dtype="bf16x3")
                    except stl.StencilError:
                        continue
                    made += 1
                    assert d == 2
                    for t in range(1, T + 1):
                        assert stl.kernel_available("mfma", "bf16x3", shape, d, r, t), (shape, r, T, t)
    assert made >= 24
