"""The lanes of the synchronisation and the write pass on the kernels' own tables (sync_span, write_span and their _rst forms)
against the plain lanes that take one symbol after the other from the tables of jpgd_lut.h, on the CPU: exact."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import jpegfile as jf
from oracle import OracleImage
from workloads import encode_jpeg, small_image

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EMUL_DIR = os.path.join(ROOT, "tests", "emul")


@pytest.fixture(scope="module")
def lanes():
    lib_path, src = os.path.join(EMUL_DIR, "libjpgd_sync.so"), os.path.join(EMUL_DIR, "jpgd_sync.cpp")
    csrc = os.path.join(ROOT, "paper_2111_09219_amd", "csrc")
    deps = [src] + [os.path.join(EMUL_DIR, f) for f in os.listdir(EMUL_DIR) if f.endswith(".h")] + [os.path.join(csrc, f) for f in os.listdir(csrc)]
    if not os.path.exists(lib_path) or any(os.path.getmtime(d) > os.path.getmtime(lib_path) for d in deps):
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", lib_path, src,
                               os.path.join(csrc, "jpgd_parse.cpp")])
    lib = ctypes.CDLL(lib_path)
    vp, u32 = ctypes.c_void_p, ctypes.c_uint32
    lib.sync_vs_plain.argtypes = [vp, ctypes.c_size_t, u32, u32, u32, u32, u32, vp]
    lib.write_vs_plain.argtypes = [vp, ctypes.c_size_t, u32, u32, ctypes.c_int, u32, u32, u32, vp]
    lib.sync_table_vs_lut.argtypes = [vp, vp, ctypes.c_int]
    lib.walk_vs_lanes.argtypes = [vp, ctypes.c_size_t, u32, u32, u32, u32, vp, vp]
    lib.lanes_restarted.argtypes = [vp, ctypes.c_size_t, u32, u32, u32, vp]
    return lib


@pytest.mark.parametrize("sub,opt,q,shape,L,ri,org", [
    ("420", False, 92, (137, 251), 128, 0, 0), ("444", True, 75, (96, 120), 1024, 0, 4096), ("gray", False, 30, (200, 64), 256, 0, 32),
    ("422", True, 98, (64, 80), 512, 0, 1 << 20), ("420", True, 10, (160, 160), 128, 0, 0), ("444", False, 100, (64, 64), 2048, 0, 64),
    ("420", True, 95, (96, 160), 256, 1, 0), ("422", False, 60, (120, 96), 128, 3, 1 << 20), ("gray", True, 90, (64, 200), 1024, 25, 96),
    # positions counted from the middle of the stream: org is negative, modulo 2^32
    ("420", False, 92, (137, 251), 128, 0, (1 << 32) - 512), ("420", True, 85, (137, 251), 128, 9, (1 << 32) - 512)])
def test_lanes_equal_the_plain_ones_from_any_state(lanes, sub, opt, q, shape, L, ri, org):
    """Position, unit, zig-zag index, unit count, DC sums and "an interval began" after every subsequence, from random
    states most of which do not lie on the true chain."""
    data = encode_jpeg(small_image(21, shape[0], shape[1], sigma=14.0), q, sub, opt, ri).data
    n = ctypes.c_uint32()
    assert lanes.sync_vs_plain(data.ctypes.data, data.size, L, 4000, 5, org, 3, ctypes.byref(n)) == 0
    assert n.value > 3000


@pytest.mark.parametrize("sub,opt,q,shape,L,ri,org,total", [
    ("420", False, 92, (137, 251), 128, 0, 0, 0), ("444", True, 75, (96, 120), 1024, 0, 4096, 0), ("gray", False, 30, (200, 64), 256, 0, 32, 100),
    ("422", True, 98, (64, 80), 512, 0, 1 << 20, 0), ("444", False, 100, (64, 64), 2048, 0, 64, 0), ("420", True, 10, (160, 160), 128, 0, 0, 301),
    ("420", True, 95, (96, 160), 256, 1, 0, 0), ("422", False, 60, (120, 96), 128, 3, 1 << 20, 0), ("gray", True, 90, (64, 200), 1024, 25, 96, 0),
    ("444", True, 85, (96, 160), 128, 5, (1 << 32) - 512, 250)])
@pytest.mark.parametrize("chain", [1, 0])
def test_write_lanes_equal_the_plain_ones(lanes, sub, opt, q, shape, L, ri, org, total, chain):
    """Stores in their order, unit, position, state, predictors and flags, on the true chain and from random states (where
    symbols run past their unit and bits start no codeword); also where the image's units end inside a subsequence."""
    data = encode_jpeg(small_image(21, shape[0], shape[1], sigma=14.0), q, sub, opt, ri).data
    n = ctypes.c_uint32()
    assert lanes.write_vs_plain(data.ctypes.data, data.size, L, 4000, chain, org, total, 3, ctypes.byref(n)) == 0
    assert n.value > 200


def _constant_dc(shape):
    """Data units whose mean is 128: every DC difference is zero, and the optimised DC table has a single codeword."""
    px = np.random.default_rng(4).normal(0, 20, (shape[0] // 8, 8, shape[1] // 8, 8))
    px -= px.mean(axis=(1, 3), keepdims=True)
    return np.clip(np.rint(px + 128), 0, 255).astype(np.uint8).reshape(shape)


@pytest.mark.parametrize("sub,opt,q", [("420", False, 92), ("444", True, 75), ("422", True, 98), ("gray", True, 30)])
def test_position_unit_and_index_say_all_about_a_lane(lanes, sub, opt, q):
    """Chains move from lane to lane and are compared by these three alone, so nothing else may decide what a lane reads next,
    also behind bits that start no codeword (in front of a coefficient, or of a DC value, of which a table of one codeword
    has many)."""
    px = _constant_dc((160, 200)) if sub == "gray" else small_image(21, 96, 160, sigma=14.0)
    data = encode_jpeg(px, q, sub, opt).data
    n = ctypes.c_uint32()
    assert lanes.lanes_restarted(data.ctypes.data, data.size, 3000, 40, 7, ctypes.byref(n)) == 0
    assert n.value > 50000


# tables of the three components and the kinds of data units they make: one pair, two, a component with a pair of its own in four
# tables (which are all a baseline file may have; also one class with three of them) and in six
PAIRINGS = [((0, 0, 0), (1, 1, 1), 1), ((0, 1, 1), (0, 1, 1), 2), ((0, 1, 0), (0, 1, 1), 3), ((1, 1, 0), (0, 1, 1), 3),
            ((0, 0, 0), (0, 1, 2), 3), ((0, 1, 2), (1, 1, 1), 3), ((0, 1, 2), (0, 1, 2), 3), ((0, 1, 0), (0, 1, 0), 2)]


@pytest.mark.parametrize("td,ta,kinds", PAIRINGS)
@pytest.mark.parametrize("sub,q,L", [("420", 90, 128), ("444", 60, 1024), ("422", 97, 256)])
def test_walk_equals_the_lanes_for_every_pairing_of_tables(lanes, td, ta, kinds, sub, q, L):
    """The walk of a whole wavefront knows the image's data units by the word the host makes of them; whatever tables the
    components share, it must take the symbols a lane takes."""
    data = jf.written_with_tables(encode_jpeg(small_image(33, 96, 144, sigma=16.0), q, sub), td, ta)
    n, k = ctypes.c_uint32(), ctypes.c_uint32()
    assert lanes.walk_vs_lanes(data.ctypes.data, data.size, L, 1500, 4, 5, ctypes.byref(n), ctypes.byref(k)) == 0
    assert n.value > 1000 and k.value == kinds


def test_tables_hold_what_the_first_ones_hold(lanes):
    """Every 16-bit stretch: bits taken, slots, value bits; tables with codes of up to 16 bits in both classes."""
    px = np.full((256, 256, 3), 128, np.uint8)
    px[::37, ::41] = (255, 0, 90)
    tables = []
    for data in (encode_jpeg(small_image(8, 160, 160, sigma=30), 97, "420", False).data,
                 encode_jpeg(small_image(8, 160, 160, sigma=30), 97, "420", True).data, encode_jpeg(px, 100, "444", True).data):
        img = OracleImage(data)
        for cls in (0, 1):
            for tid in (0, 1):
                bits, vals = img.huffman(cls, tid)
                tables.append((np.array(bits, np.uint8), np.array(vals, np.uint8), cls == 0))
    # DC codes of 10 to 16 bits, in and behind the first half of a 9-bit prefix; a table of one code; an AC table of long codes
    for counts in ([1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1], [0, 2, 1, 1, 1, 1, 1, 0, 0, 3, 0, 1, 0, 0, 0, 1], [1, 1, 1, 1, 1, 0, 1, 1, 0, 0, 0, 0, 0, 0, 0, 5], [1]):
        bits = np.array(counts + [0] * (16 - len(counts)), np.uint8)
        tables.append((bits, np.arange(bits.sum(), dtype=np.uint8), True))
    tables.append((np.array([0] * 10 + [40, 30, 20, 10, 60, 96], np.uint8), np.arange(256, dtype=np.uint8), False))
    for bits, vals, is_dc in tables:
        v = np.zeros(256, np.uint8)
        v[:len(vals)] = vals
        bits = np.ascontiguousarray(bits)
        assert lanes.sync_table_vs_lut(bits.ctypes.data, v.ctypes.data, int(is_dc)) == 0
