"""Registers of the built score kernels, from the resource notes of the library: none of the key-stationary
kernels spills, and each fits the waves per SIMD that it is made for (512 registers a lane and SIMD, in eights)."""
import re
import struct
import subprocess

import pytest

import paper_2509_05165_amd as kv


def _code_objects(data):
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", -1
    while (at := data.find(magic, at + 1)) >= 0:
        count, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                yield data[at + off:at + off + size]
            p += 24 + length


def _unpack(b, p=0):
    """The value at b[p:] in MessagePack, as far as the notes use it, and what follows it."""
    t = b[p]
    if t < 0x80:
        return t, p + 1
    if t in (0xc0, 0xc2, 0xc3):
        return {0xc0: None, 0xc2: False, 0xc3: True}[t], p + 1
    if 0xcc <= t <= 0xcf or 0xd0 <= t <= 0xd3:
        n = 1 << (t & 3)
        return int.from_bytes(b[p + 1:p + 1 + n], "big", signed=t >= 0xd0), p + 1 + n
    if 0xa0 <= t < 0xc0 or 0xd9 <= t <= 0xdb:
        w = 0 if t < 0xc0 else 1 << (t - 0xd9)
        n = t & 31 if not w else int.from_bytes(b[p + 1:p + 1 + w], "big")
        return b[p + 1 + w:p + 1 + w + n].decode(), p + 1 + w + n
    w = {0xdc: 2, 0xdd: 4, 0xde: 2, 0xdf: 4}.get(t, 0)
    n, p = (int.from_bytes(b[p + 1:p + 1 + w], "big") if w else t & 15), p + 1 + w
    out = []
    is_map = t < 0x90 or t >= 0xde
    for _ in range(2 * n if is_map else n):
        v, p = _unpack(b, p)
        out.append(v)
    return (dict(zip(out[::2], out[1::2])) if is_map else out), p


def _notes(elf):
    sections, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for at in range(sections, sections + size * count, size):
        if struct.unpack_from("<I", elf, at + 4)[0] == 7:                 # SHT_NOTE
            p, length = struct.unpack_from("<QQ", elf, at + 24)
            end = p + length
            while p < end:
                name, desc, kind = struct.unpack_from("<III", elf, p)
                p += 12 + (name + 3) // 4 * 4
                if kind == 32:                                            # NT_AMDGPU_METADATA
                    yield _unpack(elf[p:p + desc])[0]
                p += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    data = open(kv.lib_path(), "rb").read()
    found = [k for elf in _code_objects(data) for note in _notes(elf) for k in note["amdhsa.kernels"]]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), text=True, capture_output=True,
                           check=True).stdout.splitlines()
    return dict(zip(names, found))


def _fits(kernel, waves):
    return kernel[".vgpr_spill_count"] == 0 and (kernel[".vgpr_count"] + 7) // 8 * 8 * waves <= 512


def test_key_stationary_kernels(kernels):
    seen = 0
    for name, k in kernels.items():
        m = re.search(r"score_tile<(float|unsigned short), (\d+), (true|false), (true|false)>", name)
        if m:
            ks = int(m.group(2))
            assert _fits(k, 1 if ks > 16 else 2 if ks > 8 else 3 if ks > 5 else 4), m.group(0)
            seen += 1
    assert seen == 3 * 9


def test_key_stationary_emit_pass_of_the_query_stationary_shapes(kernels):
    found = [k for name, k in kernels.items() if "score_emit_keys<" in name]
    assert len(found) == 2 and all(_fits(k, 3) for k in found)
