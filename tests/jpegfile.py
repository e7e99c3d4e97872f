"""Hand assembly of small baseline JPEG files for tests: explicit tables, explicit scan bits.

Nothing here decodes anything; it only writes marker segments and packs bit strings, so
tests can feed the oracle and the library streams whose content is known by construction.
"""
from __future__ import annotations

import struct

import numpy as np


def seg(marker: int, payload: bytes) -> bytes:
    return struct.pack(">BBH", 0xFF, marker, len(payload) + 2) + payload


def dqt(tid: int, table_zigzag) -> bytes:
    return seg(0xDB, bytes([tid]) + bytes(int(v) for v in table_zigzag))


def dht(cls: int, tid: int, bits, vals) -> bytes:
    assert len(bits) == 16 and sum(bits) == len(vals)
    return seg(0xC4, bytes([(cls << 4) | tid]) + bytes(bits) + bytes(vals))


def sof0(width: int, height: int, comps) -> bytes:
    """comps: list of (id, h, v, tq)"""
    body = struct.pack(">BHHB", 8, height, width, len(comps))
    for cid, h, v, tq in comps:
        body += bytes([cid, (h << 4) | v, tq])
    return seg(0xC0, body)


def sos(comps) -> bytes:
    """comps: list of (id, td, ta)"""
    body = bytes([len(comps)])
    for cid, td, ta in comps:
        body += bytes([cid, (td << 4) | ta])
    return seg(0xDA, body + bytes([0, 63, 0]))


def pack_bits(bitstring: str, pad_ones: bool = True) -> bytes:
    """'0'/'1' characters (anything else ignored) -> bytes, MSB first, last byte padded with 1s."""
    b = [c for c in bitstring if c in "01"]
    if pad_ones:
        while len(b) % 8:
            b.append("1")
    else:
        assert len(b) % 8 == 0
    return bytes(int("".join(b[i:i + 8]), 2) for i in range(0, len(b), 8))


def stuff(raw: bytes) -> bytes:
    out = bytearray()
    for v in raw:
        out.append(v)
        if v == 0xFF:
            out.append(0)
    return bytes(out)


def assemble(width, height, comps_sof, comps_sos, qtables, dhts, scan_raw: bytes, dri: int | None = None) -> np.ndarray:
    """qtables: {tid: 64 values in zig-zag order}; dhts: [(cls, tid, bits, vals)]; scan_raw: unstuffed bytes."""
    f = b"\xFF\xD8"
    for tid, t in qtables.items():
        f += dqt(tid, t)
    f += sof0(width, height, comps_sof)
    for cls, tid, bits, vals in dhts:
        f += dht(cls, tid, bits, vals)
    if dri is not None:
        f += seg(0xDD, struct.pack(">H", dri))
    f += sos(comps_sos)
    f += stuff(scan_raw)
    f += b"\xFF\xD9"
    return np.frombuffer(f, dtype=np.uint8).copy()


# Codewords of the typical luminance tables as printed in ITU-T T.81 Annex K (Tables K.3 and K.5).
# Typed in from the standard; used to write streams by hand.
K3_DC_LUMA = {0: "00", 1: "010", 2: "011", 3: "100", 4: "101", 5: "110", 6: "1110", 7: "11110", 8: "111110",
              9: "1111110", 10: "11111110", 11: "111111110"}
K5_AC_LUMA = {(0, 0): "1010", (0, 1): "00", (0, 2): "01", (0, 3): "100", (0, 4): "1011", (0, 5): "11010",
              (1, 1): "1100", (1, 2): "11011", (2, 1): "11100", (3, 1): "111010", (4, 1): "111011",
              (15, 0): "11111111001"}


def value_bits(v: int) -> tuple[int, str]:
    """(size, bits) of a coefficient in JPEG's sign convention: negative v -> v + 2^size - 1."""
    if v == 0:
        return 0, ""
    size = abs(v).bit_length()
    raw = v if v > 0 else v + (1 << size) - 1
    return size, format(raw, "0%db" % size)


# ---- header surgery on files another encoder wrote (the entropy-coded data stays as it is) ----------------

def _segments(b: bytes):
    """(offset, marker, length field) of every segment up to and including SOS."""
    i = 2
    while i < len(b):
        assert b[i] == 0xFF
        mk, ln = b[i + 1], (b[i + 2] << 8) | b[i + 3]
        yield i, mk, ln
        if mk == 0xDA:
            return
        i += 2 + ln


def with_tables_of_its_own_for_the_third_component(data: np.ndarray) -> np.ndarray:
    """A three-component file whose second and third components share tables 1/1 becomes one whose third component
    uses tables 2/2, copies of 1/1: the same coefficients, but three DC and three AC tables to keep apart."""
    b = bytearray(np.asarray(data, np.uint8).tobytes())
    tabs, sos_at = {}, None
    for at, mk, ln in _segments(bytes(b)):
        if mk == 0xC4:
            j = at + 4
            while j < at + 2 + ln:
                n = sum(b[j + 1:j + 17])
                tabs[b[j]] = (bytes(b[j + 1:j + 17]), bytes(b[j + 17:j + 17 + n]))
                j += 17 + n
        if mk == 0xDA:
            sos_at = at
    extra = b""
    for cls in (0, 1):
        bits, vals = tabs[(cls << 4) | 1]
        extra += seg(0xC4, bytes([(cls << 4) | 2]) + bits + vals)
    assert b[sos_at + 4] == 3 and b[sos_at + 5 + 2 * 2 + 1] == 0x11
    b[sos_at + 5 + 2 * 2 + 1] = 0x22
    return np.frombuffer(bytes(b[:sos_at]) + extra + bytes(b[sos_at:]), np.uint8).copy()


def relabelled_as_1x2(data: np.ndarray) -> np.ndarray:
    """A 4:2:2 file (luma sampled 2x1: MCUs of 16x8 pixels) re-labelled as one with luma sampled 1x2 (MCUs of 8x16)
    and the frame size that gives the same grid of MCUs: the scan is the same sequence of data units, so the
    coefficients are the same, while the pixels are laid out for the new geometry."""
    b = bytearray(np.asarray(data, np.uint8).tobytes())
    for at, mk, ln in _segments(bytes(b)):
        if mk == 0xC0:
            h, w = (b[at + 5] << 8) | b[at + 6], (b[at + 7] << 8) | b[at + 8]
            mx, my = -(-w // 16), -(-h // 8)
            b[at + 5:at + 7] = (my * 16).to_bytes(2, "big")
            b[at + 7:at + 9] = (mx * 8).to_bytes(2, "big")
            assert b[at + 11] == 0x21
            b[at + 11] = 0x12
    return np.frombuffer(bytes(b), np.uint8).copy()


def written_with_tables(enc, td, ta) -> np.ndarray:
    """The scan of an encoded three-component file (workloads.EncodedJpeg with its coefficients, without restart intervals,
    typical tables) written once more with other tables: component c takes DC table td[c] and AC table ta[c], where 0 and 1
    are the file's own and 2 and 3 copies of 1.  The same coefficients."""
    b = np.asarray(enc.data, np.uint8).tobytes()
    tabs, sos_at, sampling = {}, None, None
    for at, mk, ln in _segments(b):
        if mk == 0xC4:
            j = at + 4
            while j < at + 2 + ln:
                n = sum(b[j + 1:j + 17])
                tabs[(b[j] >> 4, b[j] & 15)] = (b[j + 1:j + 17], b[j + 17:j + 17 + n])
                j += 17 + n
        if mk == 0xC0:
            sampling = b[at + 11]
        if mk == 0xDA:
            sos_at = at
    extra = b""
    for cls in (0, 1):
        for tid in (2, 3):
            tabs[(cls, tid)] = tabs[(cls, 1)]
            if tid in (td, ta)[cls]:
                extra += dht(cls, tid, *tabs[(cls, tid)])
    luma = (sampling >> 4) * (sampling & 15)
    coef = enc.coef.astype(np.int64)
    n = coef.shape[0]
    comp = np.tile([0] * luma + [1, 2], n // (luma + 2))
    unit_diff = np.zeros(n, np.int64)
    for c in range(3):
        unit_diff[comp == c] = np.diff(coef[comp == c, 0], prepend=0)
    # symbols in order: unit, zig-zag index, runs of sixteen zeros in front of a coefficient
    uu, zz = np.nonzero(coef[:, 1:])
    zz = zz + 1
    first = np.diff(uu, prepend=-1) != 0
    run = zz - np.where(first, 0, np.concatenate([[0], zz[:-1]])) - 1
    zrl = run >> 4
    last = np.zeros(n, np.int64)
    np.maximum.at(last, uu, zz)
    eob = np.flatnonzero(last < 63)
    of = np.repeat(np.arange(uu.size), zrl)          # coefficient that a run of sixteen belongs to
    nth = np.arange(of.size) - np.repeat(np.cumsum(zrl) - zrl, zrl)
    unit = np.concatenate([np.arange(n), uu, uu[of], eob])
    order = np.concatenate([np.zeros(n, np.int64), zz * 8 + 7, zz[of] * 8 + nth, np.full(eob.size, 64 * 8)])
    value = np.concatenate([unit_diff, coef[uu, zz], np.zeros(of.size + eob.size, np.int64)])
    cls = np.concatenate([np.zeros(n, np.int64), np.ones(uu.size + of.size + eob.size, np.int64)])
    size = np.where(value == 0, 0, np.floor(np.log2(np.maximum(np.abs(value), 1))).astype(np.int64) + 1)
    symbol = np.concatenate([size[:n], (run & 15) << 4, np.full(of.size, 0xF0), np.zeros(eob.size, np.int64)])
    symbol[n:n + uu.size] |= size[n:n + uu.size]
    table = np.where(cls == 0, np.asarray(td)[comp[unit]], np.asarray(ta)[comp[unit]])
    code, length = np.zeros((2, 4, 256), np.int64), np.zeros((2, 4, 256), np.int64)
    for (k, tid), (bits, vals) in tabs.items():
        next_code, at = 0, 0
        for ln in range(1, 17):
            for v in vals[at:at + bits[ln - 1]]:
                code[k, tid, v], length[k, tid, v] = next_code, ln
                next_code += 1
            at += bits[ln - 1]
            next_code <<= 1
    k = np.lexsort((order, unit))
    cls, table, symbol, value, size = cls[k], table[k], symbol[k], value[k], size[k]
    assert (length[cls, table, symbol] > 0).all()
    word = (code[cls, table, symbol] << size) | np.where(value < 0, value + (1 << size) - 1, value)
    total = length[cls, table, symbol] + size
    end = np.cumsum(total)
    bits = np.ones(int(end[-1] + 7) // 8 * 8, np.uint8)
    for j in range(int(total.max())):
        on = total > j
        bits[(end - total + j)[on]] = (word[on] >> (total[on] - 1 - j)) & 1
    raw = np.packbits(bits)
    scan = np.insert(raw, np.flatnonzero(raw == 0xFF) + 1, 0).astype(np.uint8)
    head = bytearray(b[:sos_at] + extra + b[sos_at:enc.scan_offset])
    for c in range(3):
        head[sos_at + len(extra) + 6 + 2 * c] = td[c] << 4 | ta[c]
    return np.concatenate([np.frombuffer(bytes(head), np.uint8), scan, np.array([0xFF, 0xD9], np.uint8)])
