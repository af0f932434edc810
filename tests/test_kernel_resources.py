"""Scratch memory of the kernels as built: read from the code objects' metadata in the library (no GPU)."""
import struct

import msgpack
import pytest


def _kernels(path):
    """name -> metadata of every gfx950 kernel of the library: the AMDGPU ELF files inside it, their notes' msgpack."""
    data = open(path, "rb").read()
    out, at = {}, 0
    while (at := data.find(b"\x7fELF\x02", at + 1)) > 0:   # (not the library itself at 0)
        if struct.unpack_from("<H", data, at + 18)[0] != 224:          # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", data, at + 40)
        entsize, count = struct.unpack_from("<HH", data, at + 58)
        for i in range(count):
            head = at + shoff + i * entsize
            kind, = struct.unpack_from("<I", data, head + 4)
            off, size = struct.unpack_from("<QQ", data, head + 24)
            if kind != 7:                                  # SHT_NOTE
                continue
            p, end = at + off, at + off + size
            while p < end:
                n_name, n_desc, note = struct.unpack_from("<III", data, p)
                desc = p + 12 + (n_name + 3) // 4 * 4
                if note == 32:                             # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(data[desc:desc + n_desc]).get("amdhsa.kernels", []):
                        out[k[".name"]] = k
                p = desc + (n_desc + 3) // 4 * 4
    return out


@pytest.fixture(scope="module")
def kernels(lib):
    return _kernels(lib.LIB_PATH)


@pytest.mark.parametrize("name,least", [("attn_bf16_kernel", 36), ("attn_merge_kernel", 1), ("attn_f32_wide_kernel", 3),
                                        ("embed_norm_kernel", 4), ("", 300)])
def test_kernels_keep_what_is_in_flight_in_registers(kernels, name, least):
    """Every instance: what a kernel requests ahead (attention: the next block's K and V through the softmax) fits beside what it
    works on."""
    of = {k: v for k, v in kernels.items() if name in k}
    assert len(of) >= least
    assert {k: v[".private_segment_fixed_size"] for k, v in of.items() if v[".private_segment_fixed_size"]} == {}
