"""The registers of the built convolution kernels, read from the library's own code objects (no GPU).

A compute unit's four SIMDs have 512 vector registers per lane each, ordinary and accumulation registers together: a kernel of
at most 256 leaves a SIMD two waves, of at most 168 three.  How many workgroups share a compute unit is what the tile rules count on, and
nothing else would show when an edit or a compiler takes a kernel over such an edge."""
import os
import re
import struct

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1903_12650_amd", "librn50_hip.so")


def _section(elf, name):
    start, = struct.unpack_from("<Q", elf, 0x28)
    size, count, strings = struct.unpack_from("<HHH", elf, 0x3A)
    header = lambda i: struct.unpack_from("<IIQQQQ", elf, start + i * size)
    names = header(strings)[4]
    for i in range(count):
        h = header(i)
        at = names + h[0]
        if elf[at:elf.index(b"\0", at)].decode() == name:
            return elf[h[4]:h[4] + h[5]]
    raise AssertionError("no section " + name)


def _decode(b, p):
    """One msgpack value (the kinds that kernel metadata holds) at b[p:], and where the next one starts."""
    t = b[p]
    p += 1
    if t <= 0x7F or t >= 0xE0:
        return (t if t <= 0x7F else t - 256), p
    if t in (0xC0, 0xC2, 0xC3):
        return {0xC0: None, 0xC2: False, 0xC3: True}[t], p
    if 0xCC <= t <= 0xCF:
        n = 1 << (t - 0xCC)
        return int.from_bytes(b[p:p + n], "big"), p + n
    if 0xD0 <= t <= 0xD3:
        n = 1 << (t - 0xD0)
        return int.from_bytes(b[p:p + n], "big", signed=True), p + n
    kind, n = {0x8: ("map", t & 15), 0x9: ("list", t & 15), 0xA: ("str", t & 31), 0xB: ("str", t & 31)}.get(t >> 4, (None, 0))
    if kind is None:
        kind, width = {0xD9: ("str", 1), 0xDA: ("str", 2), 0xDB: ("str", 4), 0xDC: ("list", 2), 0xDD: ("list", 4), 0xDE: ("map", 2), 0xDF: ("map", 4)}[t]
        n, p = int.from_bytes(b[p:p + width], "big"), p + width
    if kind == "str":
        return b[p:p + n].decode(), p + n
    out = []
    for _ in range(n * (2 if kind == "map" else 1)):
        v, p = _decode(b, p)
        out.append(v)
    return (dict(zip(out[::2], out[1::2])) if kind == "map" else out), p


def _kernels():
    """The metadata of every kernel: one code object per source file, bundled in a section of the library."""
    bundles, magic, at, found = _section(open(LIB, "rb").read(), ".hip_fatbin"), b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (at := bundles.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", bundles, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", bundles, p)
            target = bundles[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" not in target:
                continue
            note, q = _section(bundles[at + offset:at + offset + size], ".note"), 0
            while q < len(note):
                name, desc, kind = struct.unpack_from("<III", note, q)
                q += 12 + (name + 3 & ~3)
                if kind == 32:
                    found += _decode(note, q)[0]["amdhsa.kernels"]
                q += desc + 3 & ~3
        at += len(magic)
    return found


IGEMM = re.compile(r"igemm_kernelI([ft])" + "Li([0-9]+)E" * 5 + "Lb([01])ELb([01])ELi([0-9])ELb([01])E")


def _convolutions():
    """(element type, rows, columns, waves along rows, along columns, mode, linear, input BN, taps, written through) -> metadata."""
    out = {}
    for k in _kernels():
        m = IGEMM.search(k[".name"])
        if m:
            out[("f32" if m.group(1) == "f" else "bf16",) + tuple(int(g) for g in m.groups()[1:])] = k
    assert len(out) >= 200, len(out)
    return out


@pytest.fixture(scope="module")
def convolutions():
    return _convolutions()


def test_every_tile_leaves_a_simd_two_waves_and_keeps_its_values_in_registers(convolutions):
    """(.vgpr_count counts accumulation registers too; a few bytes of a lane's private memory are scalar registers')"""
    bad = {key: (k[".vgpr_count"], k[".agpr_count"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for key, k in convolutions.items()
           if k[".vgpr_count"] > 256 or k[".agpr_count"] or k[".vgpr_spill_count"] or k[".private_segment_fixed_size"] > 32}
    assert not bad, bad


def test_data_gradients_without_sums_do_not_hold_the_operands_of_the_sums(convolutions):
    """Their short reductions are bound by registers, not LDS: 128x128 tiles three waves per SIMD, smaller ones four (by filter rows three)."""
    most = {}
    for (dt, bm, bn, wm, wn, mode, lin, _, taps, through), k in convolutions.items():
        if mode == 3 and (wm, wn) == (2, 2) and not (bm == 128 and taps):
            key = (bm, bn, taps == 3)
            most[key] = max(most.get(key, 0), k[".vgpr_count"])
    assert set(most) == {(64, 64, False), (64, 64, True), (128, 64, False), (128, 128, False)}
    assert most[(64, 64, False)] <= 128 and most[(128, 64, False)] <= 128 and most[(64, 64, True)] <= 168 and most[(128, 128, False)] <= 168, most


def test_tiles_whose_lds_is_counted_to_the_byte(convolutions):
    """128x128 tiles that count on two or three workgroups per compute unit have no static LDS beside what their launch asks for; the bf16 forward one counts on
    three, so on three waves per SIMD (its two buffers of one operand and one of the other are 48 KB)."""
    lean = 0
    for (dt, bm, bn, wm, wn, mode, lin, in_bn, taps, through), k in convolutions.items():
        if (bm, bn, wm, wn) != (128, 128, 2, 2) or in_bn:
            continue
        if taps or mode in (0, 2):
            assert k[".group_segment_fixed_size"] == 0, (dt, mode, lin, taps)
        if dt == "bf16" and mode == 0 and not taps:
            lean += 1
            assert k[".vgpr_count"] <= 168, (lin, k[".vgpr_count"])
    assert lean == 2
