"""The kernels at the edges of their tiles and dispatch rules, against the CPU oracle: coefficients bit-exact, pixels
within one level (fp32 against double, the bound of test_gpu_parity.py)."""
import numpy as np
import pytest

import paper_2111_09219_amd as J
from oracle import OracleImage, unstuff_bytes
from workloads import encode_jpeg, small_image

import jpegfile as jf

pytestmark = pytest.mark.gpu


def _check(batch, i, data, pixels=True):
    o = OracleImage(data)
    ref = o.coefficients()
    assert np.array_equal(batch.coefficients(i).cpu().numpy(), ref)
    if pixels:
        d = np.abs(batch.pixels(i).cpu().numpy().astype(np.int16) - o.pixels(ref).astype(np.int16))
        assert d.max() <= 1
    return o


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 4095, 4096, 4097, 8191, 8192, 65537, 256 * 4096 - 1, 256 * 4096, 256 * 4096 + 1])
@pytest.mark.parametrize("share", [0.0, 0.004, 0.3, 1.0])
def test_unstuffing_at_tile_edges(n, share):
    """n stuffed bytes, a given share of them 0xFF or the zero behind it: lanes, wavefronts and tiles that begin and end
    inside a pair, a word, a 16-byte store; up to and beyond the 256 tiles a workgroup sums by itself."""
    import torch
    rng = np.random.default_rng(n + int(share * 1000))
    raw = rng.integers(0, 255, n, dtype=np.uint8)                     # no 0xFF
    raw[rng.random(n) < 0.02] = 0                                     # zeros that stay
    at = np.flatnonzero(rng.random(n - 1) < share / 2 + (share == 1.0)) if n > 1 else np.zeros(0, np.int64)
    at = at[np.concatenate([[True], np.diff(at) > 1])] if at.size and share < 1.0 else at[::2]
    raw[at] = 255
    raw[at + 1] = 0
    want = unstuff_bytes(raw)
    assert want.size == n - at.size
    d_in = torch.zeros((n + 15) // 16 * 16, dtype=torch.uint8)
    d_in[:n] = torch.from_numpy(raw)
    d_out = torch.full((n + 512,), 0xAA, dtype=torch.uint8, device="cuda")
    ws = torch.empty(4096 + 4 * (n // 4096 + 2), dtype=torch.uint8, device="cuda")
    k = J.jpgd_unstuff(d_in.cuda()[:n], d_out, ws)
    got = d_out.cpu().numpy()
    assert k == want.size and np.array_equal(got[:k], want)
    assert not got[k:k + 192].any() and (got[k + 192:] == 0xAA).all()


def _kernels_of_unstuffing(batch, data):
    """Decodes twice in a row on the same buffers, checks both, returns (kernels that only count, tiles)."""
    for _ in range(2):
        batch.d_workspace.fill_(0xA5)
        rep = batch.decode()
        _check(batch, 0, data)
    return rep.as_dict()["launches"]["unstuff_count"], -(-batch.infos[0].scan_bytes // 4096)


@pytest.mark.parametrize("side", [16, 120, 176, 280, 282, 284, 286, 290, 400])
def test_single_images_around_the_one_kernel_unstuffing(side):
    """Calls with one image of 1 to about 32 tiles: up to 16 are unstuffed by one kernel, which also copies the parameters
    while other workgroups write the image state; twice in a row on the same buffers."""
    data = encode_jpeg(small_image(side, side, side, ncomp=1, sigma=25.0), 97, "gray").data
    counted, tiles = _kernels_of_unstuffing(J.prepare_batch([data], J.Config.make()), data)
    assert counted == (0 if tiles <= 16 else 1)
    assert (tiles > 16) == (side > 280)                                # both ways are taken


@pytest.mark.parametrize("n,counted", [(16 * 4096 - 1, 0), (16 * 4096, 0), (16 * 4096 + 1, 1)])
def test_one_kernel_unstuffing_at_its_last_byte(n, counted):
    """A scan of sixteen full tiles and one byte more or less: filled up with bytes behind the last data unit."""
    data = encode_jpeg(small_image(276, 276, 276, ncomp=1, sigma=25.0), 97, "gray").data
    fill = n - J.jpgd_parse(data).scan_bytes
    assert fill > 0 and bytes(data[-2:]) == b"\xff\xd9"
    data = np.concatenate([data[:-2], np.full(fill, 0x55, np.uint8), data[-2:]])
    batch = J.prepare_batch([data], J.Config.make())
    assert batch.infos[0].scan_bytes == n
    assert _kernels_of_unstuffing(batch, data)[0] == counted


@pytest.mark.parametrize("sub", ["gray", "444", "422", "420"])
@pytest.mark.parametrize("w,h", [(1, 1), (7, 9), (8, 8), (9, 17), (23, 5), (31, 33), (47, 16), (100, 3), (129, 24), (130, 25), (131, 31), (385, 8), (395, 15)])
def test_pixel_rows_of_any_length(sub, w, h):
    """Groups of eight pixels cut off at the right, rows that begin at any byte, runs of MCUs that end inside a row; as RGB
    and as planes."""
    data = encode_jpeg(small_image(w * 1000 + h, h, w, ncomp=1 if sub == "gray" else 3, sigma=12.0), 90, sub).data
    batch = J.prepare_batch([data], J.Config.make())
    batch.d_pixels.fill_(0x5A)
    batch.decode()
    o = _check(batch, 0, data)
    used = h * w * (1 if sub == "gray" else 3)
    assert bool((batch.d_pixels[used:] == 0x5A).all())
    batch = J.prepare_batch([data], J.Config.make(flags=J.F_PLANAR))
    batch.decode()
    for got, ref in zip(batch.planes(0), o.planes(o.coefficients())):
        assert np.abs(got.cpu().numpy().astype(np.int16) - ref.astype(np.int16)).max() <= 1


@pytest.mark.parametrize("flags", [0, J.F_PLANAR])
@pytest.mark.parametrize("images,per_workgroup", [(14, 2), (21, 3), (28, 4), (70, 4)])
@pytest.mark.parametrize("sub,w,h", [("444", 801, 677), ("422", 1202, 677), ("420", 801, 1353), ("gray", 2404, 677)])
def test_several_runs_per_pixel_workgroup(sub, w, h, images, per_workgroup, flags):
    """Enough images in one call that a workgroup of the pixel kernel takes two, three or four runs of MCUs (one for every
    4096 runs of the call, at most four).  Each image has 7 runs in each of 85 rows of MCUs: no multiple of those numbers,
    so that workgroups go on from one row to the next and the last one of an image is cut short.  At both ends an image
    of five runs.  With 70 images the call's coefficients and pixels exceed 256 MB, and the kernel's other variant runs."""
    a = encode_jpeg(small_image(3, h, w, ncomp=1 if sub == "gray" else 3, sigma=3.0), 60, sub).data
    b = encode_jpeg(small_image(4, 40, 50, sigma=9.0), 85, "422").data
    files = [b] + [a] * images + [b]
    batch = J.prepare_batch(files, J.Config.make(flags=flags))
    runs = [-(-i.mcus_x // (48 // i.units_per_mcu)) * i.mcus_y for i in batch.infos]
    assert runs[1] == 7 * 85 and runs[0] == 5 and min(sum(runs) // 4096, 4) == per_workgroup
    assert all(runs[1] % k for k in (2, 3, 4))
    nbytes = sum(128 * i.total_units + i.width * i.height * i.ncomp for i in batch.infos)
    assert (nbytes > 256 << 20) == (images == 70)
    batch.decode()
    shown = batch.planes if flags else lambda i: [batch.pixels(i)]
    for i in (0, 1, images + 1):
        o = _check(batch, i, files[i], pixels=False)
        ref = o.planes(o.coefficients()) if flags else [o.pixels(o.coefficients())]
        assert len(ref) == len(shown(i))
        for got, want in zip(shown(i), ref):
            want = want.reshape(got.shape)
            assert np.abs(got.cpu().numpy().astype(np.int16) - want.astype(np.int16)).max() <= 1
    first = shown(1)
    for i in range(2, images + 1):
        assert all(bool((x == y).all()) for x, y in zip(shown(i), first)), i


def _canonical(lengths):
    """{symbol: code length} -> (bits, vals, {symbol: codeword})"""
    order = sorted(lengths, key=lambda s: (lengths[s], s))
    code, at, words = 0, 0, {}
    for s in order:
        code <<= lengths[s] - at
        at = lengths[s]
        words[s] = format(code, "0%db" % at)
        code += 1
    return bytes(sum(v == k for v in lengths.values()) for k in range(1, 17)), bytes(order), words


@pytest.mark.parametrize("sub", ["gray", "444", "420"])
@pytest.mark.parametrize("L", [128, 256, 1024])
def test_long_dc_and_ac_codewords(sub, L):
    """Hand-made tables in which common DC and AC symbols have codewords beyond the first-level index (11 to 16 bits), in
    the rounds with a wavefront per chain as well: coefficients and synchronisation records."""
    rng = np.random.default_rng(L)
    dc_len = {0: 2, 1: 2, 2: 3, 3: 12, 4: 11, 5: 13, 6: 14, 7: 15, 8: 16, 9: 10, 10: 9, 11: 8}
    ac_len = {0x00: 2, 0x01: 2, 0x11: 4, 0x02: 5, 0x03: 11, 0x12: 12, 0x04: 13, 0x31: 14, 0xF0: 15, 0x05: 16, 0x21: 6}
    dc2_len = dict(dc_len)
    dc2_len[3], dc2_len[11] = 8, 12
    ac2_len = {0x00: 1, 0x01: 3, 0x11: 3, 0x02: 11, 0x03: 12, 0xF0: 13, 0x21: 14}
    dc, ac, dc2, ac2 = (_canonical(t) for t in (dc_len, ac_len, dc2_len, ac2_len))
    hs = 2 if sub == "420" else 1
    units = {"gray": [0], "444": [0, 1, 2], "420": [0, 0, 0, 0, 1, 2]}[sub]
    mx, my = 40, 30
    out = []
    pred = [0, 0, 0]
    for _ in range(mx * my):
        for c in units:
            d, a, asyms = (dc[2], ac[2], list(ac_len)) if c == 0 else (dc2[2], ac2[2], list(ac2_len))
            size = int(rng.choice([0, 1, 2, 3, 4, 5, 6]))
            v = int(rng.integers(1 << (size - 1), 1 << size)) * int(rng.choice([-1, 1])) if size else 0
            if abs(pred[c] + v) > 900:
                v = -v
            pred[c] += v
            out += [d[size], jf.value_bits(v)[1]]
            z = 1
            while z < 64:
                s = int(rng.choice(asyms))
                run, n = s >> 4, s & 15
                if s == 0:
                    out.append(a[0])
                    break
                if z + run + (n == 0 and run == 15) > 63:
                    continue
                out.append(a[s])
                z += run + 1
                if n:
                    out.append(jf.value_bits(int(rng.integers(1 << (n - 1), 1 << n)) * int(rng.choice([-1, 1])))[1])
    n = 1 if sub == "gray" else 3
    sof = [(c + 1, hs if c == 0 else 1, hs if c == 0 else 1, 0) for c in range(n)]
    sos = [(c + 1, min(c, 1), min(c, 1)) for c in range(n)]
    dhts = [(0, 0, dc[0], dc[1]), (1, 0, ac[0], ac[1])] + ([] if n == 1 else [(0, 1, dc2[0], dc2[1]), (1, 1, ac2[0], ac2[1])])
    data = jf.assemble(mx * 8 * hs, my * 8 * hs, sof, sos, {0: [1] * 64}, dhts, jf.pack_bits("".join(out)))
    batch = J.prepare_batch([data], J.Config.make(subseq_bits=L))
    rep = batch.decode()
    o = _check(batch, 0, data, pixels=False)
    rec = J.jpgd_read_sync_info(batch.d_workspace, 0, rep.n_subseq + 8)
    bs = o.boundary_states(L)
    live = np.cumsum(bs["units"]) < o.total_units
    assert np.array_equal(rec["p"][live].astype(np.int64), bs["p"][live])
    assert np.array_equal(rec["u"][live], bs["u"][live]) and np.array_equal(rec["z"][live], bs["z"][live])
    assert np.array_equal(rec["units"][live], bs["units"][live])
    assert np.array_equal(rec["dcsum"][live].astype(np.int16), bs["dcsum"][live].astype(np.int16))


def _room(info, L):
    """LDS the write kernel asks for to gather its output: what the image's average workgroup covers and a quarter more."""
    units = min(info.total_units, info.total_units * 256 * L // (8 * info.scan_bytes))
    return 0 if units * 128 > 131072 else min(131072, -(-(units + units // 4 + 1) * 128 // 1024) * 1024)


def _bytes_per_workgroup(o, L):
    """Bytes of coefficients, from a 16-byte boundary on, that each workgroup of 256 subsequences covers."""
    bs = o.boundary_states(L)
    end = np.minimum(64 * np.cumsum(bs["units"]) + bs["z"], 64 * o.total_units)
    end = np.append(end[255:-1:256], 64 * o.total_units)
    begin = np.append(0, end[:-1])
    return 2 * (end - begin // 8 * 8)[end > begin]


@pytest.mark.parametrize("sub,L", [("gray", 128), ("444", 128), ("420", 256), ("422", 256)])
@pytest.mark.parametrize("quality", [5, 30, 75, 95])
@pytest.mark.parametrize("flat_rows", [0, 160])
def test_write_pass_below_and_above_its_room_in_lds(sub, L, quality, flat_rows):
    """Small calls gather a workgroup's coefficients in LDS where they fit what the call asks for: workgroups of 128 to
    about 10 000 units, in one image as well (flat rows on top of rows half flat and half noise); onto a buffer that is not
    clear."""
    px = small_image(quality, 416, 640, ncomp=1 if sub == "gray" else 3, sigma=14.0)
    px[:, :300] = 120
    px[:flat_rows] = 120
    data = encode_jpeg(px, quality, sub).data
    batch = J.prepare_batch([data], J.Config.make(subseq_bits=L))
    for _ in range(2):
        batch.d_coef.fill_(0x1234)
        batch.decode()
        o = _check(batch, 0, data)
    room, covered = _room(batch.infos[0], L), _bytes_per_workgroup(o, L)
    if quality == 95:
        assert (covered <= room).any() and ((covered > room).any() or flat_rows == 0)  # with flat rows, both ways in one call
    elif quality == 5:
        assert room == 0                                               # no workgroup gathers


@pytest.mark.parametrize("w,h,room", [(256, 256, 131072), (8 * 1024, 8, 131072), (264, 256, 0), (8 * 1025, 8, 0)])
def test_write_pass_at_the_most_room_in_lds(w, h, room):
    """One workgroup that covers 1024 data units, which fill the 128 KB exactly, or some more."""
    data = encode_jpeg(small_image(w, h, w, ncomp=1, sigma=1.0), 20, "gray").data
    batch = J.prepare_batch([data], J.Config.make(subseq_bits=256))
    batch.d_coef.fill_(0x1234)
    rep = batch.decode()
    o = _check(batch, 0, data)
    assert rep.n_subseq <= 256 and _room(batch.infos[0], 256) == room
    assert (_bytes_per_workgroup(o, 256) <= 131072).all() == (room > 0)


@pytest.mark.parametrize("images", [127, 128, 129])
@pytest.mark.parametrize("sub", ["gray", "444"])
def test_write_pass_around_the_number_of_workgroups_that_gather(images, sub):
    """Calls of 127 and 128 workgroups gather their output in LDS, one of 129 does not; images of different content."""
    files = [encode_jpeg(small_image(i, 40 + i, 70 - i % 9, ncomp=1 if sub == "gray" else 3, sigma=6.0), 50, sub).data for i in range(6)]
    files = [files[i % 6] for i in range(images)]
    batch = J.prepare_batch(files, J.Config.make(subseq_bits=128))
    assert sum(-(-i.scan_bytes * 8 // (256 * 128)) for i in batch.infos) == images
    assert max(_room(i, 128) for i in batch.infos) > 0
    batch.d_coef.fill_(0x1234)
    batch.decode()
    for i in range(images):
        if i < 6 or i > images - 6:
            _check(batch, i, files[i])
        else:
            assert bool((batch.coefficients(i) == batch.coefficients(i % 6)).all()), i


def test_gathering_write_passes_in_flight_on_four_streams():
    """Twelve small calls of different pictures and layouts at once, three per stream, beside a larger one."""
    import torch
    cases = [("gray", 256, 256, 75), ("444", 320, 240, 90), ("422", 401, 203, 85), ("444", 640, 480, 92)]
    files = [encode_jpeg(small_image(k, h, w, ncomp=1 if s == "gray" else 3, sigma=7.0), q, s).data
             for k in range(3) for s, w, h, q in cases]
    big = encode_jpeg(small_image(9, 1024, 1536, sigma=9.0), 90, "444").data
    batches = [J.prepare_batch([f], J.Config.make()) for f in files]
    large = J.prepare_batch([big] * 6, J.Config.make())
    streams = [torch.cuda.Stream() for _ in range(4)]
    for b in batches + [large]:
        b.d_coef.fill_(0x1234)
        b.d_workspace.fill_(0xA5)
    torch.cuda.synchronize()
    calls = [large.decode_async(stream=streams[0])] + [b.decode_async(stream=streams[k % 4]) for k, b in enumerate(batches)]
    for c in calls:
        J.Batch.wait(c)
    torch.cuda.synchronize()
    for b, f in zip(batches + [large], files + [big]):
        _check(b, 0, f)
