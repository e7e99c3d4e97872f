"""The decode calls this library is used for, as cases that can be timed and compared.

A case says which files are decoded (layout, size, quality, tables, restart intervals, content) and by which call;
`prepare` makes those files from a seed, on the GPU, and the buffers a program keeps beside them (`prepare_batch`);
`run` is one pass through the package's entry points and returns everything it computed: int16 coefficients and uint8
pixels.

The pictures are made here: a baseline encoder in a few tensor operations (transform, quantisation, run lengths,
Huffman codes and bit packing for all data units at once), because the largest file would keep an encoder on the host
busy for a quarter of a minute.
"""
from __future__ import annotations

import heapq
import math

import numpy as np
import torch
import torch.nn.functional as F

import paper_2111_09219_amd as J

# ------------------------------------------------------------------------------------------------ the cases

_LAYOUTS = {"gray": (1, 1, 1), "444": (3, 1, 1), "422": (3, 2, 1), "420": (3, 2, 2)}   # components, luma sampling
_FLAGS = {"rgb": 0, "planar": J.F_PLANAR, "half": J.F_SCALE_2, "quarter": J.F_SCALE_4, "eighth": J.F_SCALE_8,
          "coefficients": J.F_NO_PIXELS}
_DENOMINATOR = {"half": 2, "quarter": 4, "eighth": 8}


def _case(name, width, height, layout, quality, images=1, quality_high=None, sigma=6.0, sigma_high=None, content="photo",
          optimize=False, restart=False, output="rgb", call="decode"):
    """quality / sigma: of every image, or the low end of a range each image draws from; restart: one interval per row
    of MCUs; output: what d_pixels receives; call: "decode" (buffers kept between calls), "file" (from the file's bytes
    in host memory, buffers included) or "inflight" (one call per image, all enqueued before the first is waited for)."""
    return {"name": name, "width": width, "height": height, "layout": layout, "images": images, "quality": quality,
            "quality_high": quality if quality_high is None else quality_high, "sigma": sigma,
            "sigma_high": sigma if sigma_high is None else sigma_high, "content": content, "optimize": optimize,
            "restart": restart, "output": output, "call": call}


def listed():
    return [
        # a small gray picture on its own: a preview or a tile, where only the latency of one call counts
        _case("gray_256", 256, 256, "gray", 75, sigma=8.0),
        # one frame of video without chroma subsampling
        _case("frame_1088_444", 1920, 1088, "444", 90),
        # a noisy, finely textured picture at high quality with Huffman tables of its own (codes up to 16 bits)
        _case("square_4096_420", 4096, 4096, "420", 95, sigma=12.0, optimize=True),
        # a training or serving batch: many small pictures of different quality in one call
        _case("batch_256_420", 512, 384, "420", 70, images=256, quality_high=95, sigma=2.0, sigma_high=15.0),
        # the largest single picture: half nearly flat, half noise, so that code lengths and distances to
        # synchronise differ as much as they can inside one scan
        _case("flat_noise_16k_420", 15360, 8640, "420", 92, content="split"),
        # a batch of video frames at everyday quality: few bits per data unit, the output is most of the traffic
        _case("frames_48_444", 1920, 1088, "444", 75, images=48, sigma=4.0),
        # a camera's file: 4:2:2, one restart interval per row of MCUs, odd size, planes for further processing
        _case("camera_422_restart", 3001, 2003, "422", 88, restart=True, output="planar"),
        # thumbnails of a folder of photographs, straight from the coefficients
        _case("thumbnails_24_420", 2047, 1535, "420", 85, images=24, output="eighth"),
        # a page scanned in gray, coefficients only (transcoding)
        _case("scan_gray_coefficients", 4963, 7013, "gray", 80, sigma=3.0, optimize=True, output="coefficients"),
        # one file as it lies in host memory, odd size: headers, buffers, copy and decode in one go
        _case("file_1001_420", 1001, 667, "420", 80, sigma=4.0, call="file"),
        # photographs that arrive one by one: a call each, all in flight together on two streams
        _case("inflight_8_420", 1600, 1200, "420", 85, images=8, call="inflight"),
    ]


def draw(rng):
    """One more case of the same ranges: any layout, quality, output and call, sizes from small tiles to 16 million
    pixels a picture and 50 million a call."""
    pixels = math.exp(rng.uniform(math.log(40_000), math.log(16_000_000)))
    aspect = math.exp(rng.uniform(-0.6, 0.6))
    width = max(97, int(math.sqrt(pixels * aspect)))
    height = max(97, int(pixels / width))
    call = rng.choice(["decode", "decode", "decode", "decode", "file", "inflight"])
    most = max(1, min(256, int(50_000_000 / (width * height))))
    images = 1 if call == "file" or rng.random() < 0.4 else int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    if call == "inflight":
        images = min(max(2, images), 8)
    q = rng.randint(40, 95)
    c = _case("drawn", width, height, rng.choice(["gray", "444", "422", "420", "420"]), q, images=images,
              quality_high=min(95, q + rng.choice([0, 0, 10])), sigma=round(rng.uniform(1.0, 12.0), 2),
              content=rng.choice(["photo", "photo", "photo", "split"]), optimize=rng.random() < 0.3,
              restart=rng.random() < 0.2, output=rng.choice(["rgb"] * 5 + ["planar", "half", "quarter", "eighth", "coefficients"]),
              call=call)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ pictures

def _picture(gen, case, height, width, sigma):
    """float32 [components, height, width] in 0..255 on the generator's device."""
    dev = gen.device
    ncomp = _LAYOUTS[case["layout"]][0]

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev)

    if case["content"] == "split":
        half = width // 2
        left = 128.0 + normal(ncomp, height, half)
        right = torch.rand(ncomp, height, width - half, generator=gen, device=dev) * 255.0
        return torch.cat([left, right], dim=2).round_().clamp_(0.0, 255.0)
    img = torch.full((ncomp, height, width), 128.0, device=dev)
    # smooth shading, a few regions with sharp borders, finer texture, sensor noise
    for cells, amplitude, sharp in ((3, 45.0, False), (5, 25.0, True), (24, 12.0, False), (96, 5.0, False)):
        lattice = normal(1, ncomp, cells + 2, cells + 2)
        field = F.interpolate(lattice, size=(height, width), mode="bilinear", align_corners=True)[0]
        img += amplitude * (torch.sign(field) if sharp else field)
    img += sigma * normal(ncomp, height, width)
    return img.round_().clamp_(0.0, 255.0)


# ------------------------------------------------------------------------------------------------ the encoder
# Fixed by the standard (ITU-T T.81): the zig-zag order, the quantisation matrices of Annex K.1 and the typical Huffman
# tables of Annex K.3.

_SCAN = sorted(range(64), key=lambda i: (i // 8 + i % 8, i // 8 if (i // 8 + i % 8) % 2 else i % 8))
_K1 = [[16, 11, 10, 16, 24, 40, 51, 61, 12, 12, 14, 19, 26, 58, 60, 55, 14, 13, 16, 24, 40, 57, 69, 56, 14, 17, 22, 29, 51,
        87, 80, 62, 18, 22, 37, 56, 68, 109, 103, 77, 24, 35, 55, 64, 81, 104, 113, 92, 49, 64, 78, 87, 103, 121, 120, 101,
        72, 92, 95, 98, 112, 100, 103, 99],
       [17, 18, 24, 47, 99, 99, 99, 99, 18, 21, 26, 66, 99, 99, 99, 99, 24, 26, 56, 99, 99, 99, 99, 99, 47, 66] + [99] * 38]
_DC_BITS = [bytes.fromhex("00010501010101010100000000000000"), bytes.fromhex("00030101010101010101010000000000")]
_DC_VALS = bytes(range(12))
_AC_BITS = [bytes.fromhex("0002010303020403050504040000017d"), bytes.fromhex("00020102040403040705040400010277")]
_AC_VALS = [bytes.fromhex(
    "01020300041105122131410613516107227114328191a1082342b1c11552d1f02433627282090a161718191a25262728292a3435363738393a4344"
    "45464748494a535455565758595a636465666768696a737475767778797a838485868788898a92939495969798999aa2a3a4a5a6a7a8a9aab2b3b4"
    "b5b6b7b8b9bac2c3c4c5c6c7c8c9cad2d3d4d5d6d7d8d9dae1e2e3e4e5e6e7e8e9eaf1f2f3f4f5f6f7f8f9fa"), bytes.fromhex(
    "000102031104052131061241510761711322328108144291a1b1c109233352f0156272d10a162434e125f11718191a262728292a35363738393a43"
    "4445464748494a535455565758595a636465666768696a737475767778797a82838485868788898a92939495969798999aa2a3a4a5a6a7a8a9aab2"
    "b3b4b5b6b7b8b9bac2c3c4c5c6c7c8c9cad2d3d4d5d6d7d8d9dae2e3e4e5e6e7e8e9eaf2f3f4f5f6f7f8f9fa")]


def _quant(table, quality):
    scale = 5000 // quality if quality < 50 else 200 - 2 * quality
    return [min(255, max(1, (v * scale + 50) // 100)) for v in _K1[table]]


def _optimal(freq):
    """Code lengths for the symbols that occur (at most 16 bits, the all-ones code left out): (bits, vals)."""
    used = {s: n for s, n in enumerate(freq) if n}
    floor = 1
    while True:
        heap = [(max(n, floor), s, (s,)) for s, n in used.items()] + [(0, -1, (-1,))]
        heapq.heapify(heap)
        length = {s: 0 for s in list(used) + [-1]}
        while len(heap) > 1:
            a, b = heapq.heappop(heap), heapq.heappop(heap)
            for s in a[2] + b[2]:
                length[s] += 1
            heapq.heappush(heap, (a[0] + b[0], min(a[1], b[1]), a[2] + b[2]))
        if max(length.values()) <= 16:
            break
        floor *= 2
    deepest = max(length.values())
    order = sorted(used, key=lambda s: (length[s], s))
    if length[-1] < deepest:   # the place left out has to be the last one of the longest codes
        raise AssertionError("the rarest symbol is not among the deepest")
    return bytes(sum(length[s] == k for s in order) for k in range(1, 17)), bytes(order)


def _codes(bits, vals, dev):
    """Canonical codes of a table: code and length per symbol."""
    code, length = torch.zeros(256, dtype=torch.int64), torch.zeros(256, dtype=torch.int64)
    at = k = 0
    for n in range(1, 17):
        for _ in range(bits[n - 1]):
            code[vals[k]], length[vals[k]] = at, n
            at, k = at + 1, k + 1
        at <<= 1
    return code.to(dev), length.to(dev)


def _segment(marker, payload):
    return bytes([0xFF, marker]) + (len(payload) + 2).to_bytes(2, "big") + bytes(payload)


def _encode(img, layout, quality, optimize, restart):
    """A baseline file (bytes) of the picture img, float32 [components, height, width] (gray, or red, green, blue)."""
    dev = img.device
    ncomp, hs, vs = _LAYOUTS[layout]
    height, width = img.shape[1:]
    mx, my = -(-width // (8 * hs)), -(-height // (8 * vs))
    img = F.pad(img[None], (0, mx * 8 * hs - width, 0, my * 8 * vs - height), mode="replicate")[0]
    if ncomp == 3:
        r, g, b = img
        planes = [0.299 * r + 0.587 * g + 0.114 * b - 128.0, -0.168736 * r - 0.331264 * g + 0.5 * b,
                  0.5 * r - 0.418688 * g - 0.081312 * b]
    else:
        planes = [img[0] - 128.0]
    k = torch.arange(8, dtype=torch.float64)
    basis = 0.5 * torch.cos((2 * k[None, :] + 1) * k[:, None] * math.pi / 16)
    basis[0] *= math.sqrt(0.5)
    basis = basis.float().to(dev)
    scan = torch.tensor(_SCAN, device=dev)
    units = []
    for c, plane in enumerate(planes):
        h, v = (hs, vs) if c == 0 else (1, 1)
        if c and (hs, vs) != (1, 1):
            plane = F.avg_pool2d(plane[None, None], (vs, hs))[0, 0]
        blocks = plane.reshape(my, v, 8, mx, h, 8).permute(0, 3, 1, 4, 2, 5).reshape(-1, 8, 8)
        coef = torch.matmul(basis, torch.matmul(blocks, basis.t().contiguous())).reshape(-1, 64)
        q = torch.tensor(_quant(min(c, 1), quality), dtype=torch.float32, device=dev)
        units.append((coef / q).round_().to(torch.int16)[:, scan].reshape(mx * my, h * v, 64))
    upm = sum(u.shape[1] for u in units)
    comp = torch.tensor([0] * (hs * vs if ncomp == 3 else 1) + [1, 2][:ncomp - 1], device=dev)
    coef = torch.cat(units, dim=1).reshape(-1, 64)              # data units in scan order
    nunits = coef.shape[0]
    unit_comp = comp.repeat(mx * my)
    per_interval = mx * upm if restart else nunits
    interval_of_unit = torch.arange(nunits, device=dev) // per_interval
    for c in range(ncomp):                                      # DC differences, from zero in every interval
        idx = (unit_comp == c).nonzero()[:, 0]
        dc, part = coef[idx, 0], interval_of_unit[idx]
        before = torch.cat([dc.new_zeros(1), dc[:-1]])
        before[1:][part[1:] != part[:-1]] = 0
        coef[idx, 0] = dc - before
    # one entry per DC difference and per non-zero coefficient
    keep = coef != 0
    keep[:, 0] = True
    unit, slot = keep.nonzero().unbind(1)
    value = coef[unit, slot].to(torch.int64)
    del keep, coef
    last = torch.ones_like(unit, dtype=torch.bool)
    last[:-1] = unit[1:] != unit[:-1]
    run = torch.zeros_like(slot)
    run[1:] = slot[1:] - slot[:-1] - 1
    is_dc = slot == 0
    run[is_dc] = 0
    size = torch.frexp(value.abs().to(torch.float32))[1].to(torch.int64)     # bits of |value|; 0 for 0
    eob = last & (slot < 63)
    table = (unit_comp > 0).to(torch.int64)[unit]
    symbol = torch.where(is_dc, size, ((run & 15) << 4) | size)
    skips = run >> 4
    tables = []
    for t in range(1 if ncomp == 1 else 2):
        if optimize:
            mine = table == t
            dc = torch.bincount(symbol[mine & is_dc], minlength=256)
            ac = torch.bincount(symbol[mine & ~is_dc], minlength=256)
            ac[0] += int((mine & eob).sum())
            ac[0xF0] += int(skips[mine].sum())
            tables.append((_optimal(dc.tolist()), _optimal(ac.tolist())))
        else:
            tables.append(((_DC_BITS[t], _DC_VALS), (_AC_BITS[t], _AC_VALS[t])))
    code = torch.stack([torch.cat([_codes(*t[kind], dev)[0] for t in tables]) for kind in (0, 1)])
    length = torch.stack([torch.cat([_codes(*t[kind], dev)[1] for t in tables]) for kind in (0, 1)])
    at, kind = table * 256 + symbol, (~is_dc).to(torch.int64)
    # bits of an entry: runs of sixteen zeros, the code with its value bits, end of block
    body = (code[kind, at] << size) | ((value - (value < 0).to(torch.int64)) & ((1 << size) - 1))
    body_len = length[kind, at] + size
    eob_len = torch.where(eob, length[1, table * 256], 0)
    body = (body << eob_len) | torch.where(eob, code[1, table * 256], 0)
    body_len += eob_len
    skip_len = skips * length[1, table * 256 + 0xF0]
    del at, kind, size, symbol, eob, eob_len, last, run, slot, value
    total = skip_len + body_len
    start = total.cumsum(0) - total
    # intervals begin at a byte; the bits in front of that are ones
    interval = interval_of_unit[unit]
    nint = int(interval_of_unit[-1]) + 1
    first = torch.searchsorted(interval, torch.arange(nint, device=dev))
    begin = torch.cat([start[first], (start[-1] + total[-1])[None]])
    in_bits = begin[1:] - begin[:-1]
    in_bytes = (in_bits + 7) >> 3
    byte0 = in_bytes.cumsum(0) - in_bytes
    start += (byte0 * 8 - begin[:-1])[interval]
    nbytes = int(in_bytes.sum())
    words = torch.zeros(nbytes // 4 + 4, dtype=torch.int64, device=dev)

    def put(offset, nbits, v):                                  # up to 48 bits each; no two overlap
        word, bit = offset >> 5, offset & 31
        for j in range(3):
            shift = 32 * (j + 1) - bit - nbits
            part = torch.where(shift >= 0, v << shift.clamp(0, 31), v >> (-shift).clamp(min=0)) & 0xFFFFFFFF
            words.index_add_(0, word + j, torch.where(shift > 31, 0, part))

    put(start + skip_len, body_len, body)
    some = skips > 0
    zrl, zrl_len = code[1, table[some] * 256 + 0xF0], length[1, table[some] * 256 + 0xF0]
    n = skips[some]
    v = torch.where(n > 2, (((zrl << zrl_len) | zrl) << zrl_len) | zrl, torch.where(n > 1, (zrl << zrl_len) | zrl, zrl))
    put(start[some], n * zrl_len, v)
    pad = in_bytes * 8 - in_bits
    put(byte0 * 8 + in_bits, pad, (1 << pad) - 1)
    raw = torch.stack([(words >> s) & 255 for s in (24, 16, 8, 0)], dim=1).reshape(-1)[:nbytes].to(torch.uint8)
    # stuffing, and a marker behind every interval but the last
    full = raw == 255
    extra = full.to(torch.int64)
    ends = (byte0 + in_bytes)[:-1] - 1
    extra[ends] += 2
    to = torch.arange(nbytes, device=dev) + extra.cumsum(0) - extra
    out = torch.zeros(nbytes + int(extra.sum()), dtype=torch.uint8, device=dev)
    out[to] = raw
    mark = to[ends] + 1 + full[ends].to(torch.int64)
    out[mark] = 255
    out[mark + 1] = (0xD0 + torch.arange(nint - 1, device=dev) % 8).to(torch.uint8)
    head = b"\xff\xd8"
    for t in range(len(tables)):
        q = _quant(t, quality)
        head += _segment(0xDB, [t] + [q[i] for i in _SCAN])
    head += _segment(0xC0, [8, height >> 8, height & 255, width >> 8, width & 255, ncomp] +
                     sum([[c + 1, (hs << 4 | vs) if c == 0 and ncomp == 3 else 0x11, min(c, 1)] for c in range(ncomp)], []))
    for t, (dc, ac) in enumerate(tables):
        head += _segment(0xC4, bytes([t]) + dc[0] + dc[1]) + _segment(0xC4, bytes([16 + t]) + ac[0] + ac[1])
    if restart:
        head += _segment(0xDD, mx.to_bytes(2, "big"))
    head += _segment(0xDA, [ncomp] + sum([[c + 1, 0x11 * min(c, 1)] for c in range(ncomp)], []) + [0, 63, 0])
    return head + out.cpu().numpy().tobytes() + b"\xff\xd9"


def _files(case, seed, device, images=None, height=None, width=None):
    gen = torch.Generator(device=device).manual_seed(seed * 7919 + 17)
    spread = np.random.default_rng(seed)
    files = []
    for _ in range(case["images"] if images is None else images):
        quality = int(spread.integers(case["quality"], case["quality_high"] + 1))
        sigma = float(spread.uniform(case["sigma"], case["sigma_high"]))
        img = _picture(gen, case, height or case["height"], width or case["width"], sigma)
        files.append(_encode(img, case["layout"], quality, case["optimize"], case["restart"]))
    return files


# ------------------------------------------------------------------------------------------------ one pass

def _outputs(batch, cfg):
    return [batch.d_coef] if cfg.flags & J.F_NO_PIXELS else [batch.d_coef, batch.d_pixels]


def prepare(case, seed):
    cfg = J.Config.make(flags=_FLAGS[case["output"]])
    files = _files(case, seed, torch.device("cuda", 0))
    state = {"call": case["call"], "cfg": cfg}
    if case["call"] == "file":
        state["files"] = files
        return state
    groups = [[f] for f in files] if case["call"] == "inflight" else [files]
    state["batches"] = [J.prepare_batch(g, cfg, want_pixels=not cfg.flags & J.F_NO_PIXELS) for g in groups]
    for b in state["batches"]:
        if b.d_pixels is not None:
            b.d_pixels.zero_()      # (the bytes between two pictures, and behind a reduced one, are never written)
    if case["call"] == "inflight":
        state["streams"] = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    return state


def run(state):
    if state["call"] == "file":
        batch = J.prepare_batch(state["files"], state["cfg"], want_pixels=not state["cfg"].flags & J.F_NO_PIXELS)
        batch.decode()
        if batch.d_pixels is None:
            return [batch.d_coef]
        shown = batch.planes(0) if state["cfg"].flags & J.F_PLANAR else [batch.pixels(0)]
        return [batch.d_coef] + shown
    if state["call"] == "inflight":
        streams = state["streams"]
        calls = [b.decode_async(streams[i % len(streams)]) for i, b in enumerate(state["batches"])]
        for c in calls:
            J.Batch.wait(c)
    else:
        state["batches"][0].decode()
    return [t for b in state["batches"] for t in _outputs(b, state["cfg"])]


# ------------------------------------------------------------------------------------------------ what it takes

def work(case):
    """Bytes: the compressed scan once, the coefficients and the pixels once.  The scan's size is taken from a sample of
    the same content.  Operations: two passes of eight 8-point transforms per data unit (36 each) and the dequantisation,
    three additions or conversions per output sample; the entropy decoder's are table look-ups, one per symbol, and
    are not counted."""
    ncomp, hs, vs = _LAYOUTS[case["layout"]]
    mcus = -(-case["width"] // (8 * hs)) * -(-case["height"] // (8 * vs))
    units = mcus * (1 if ncomp == 1 else hs * vs + 2) * case["images"]
    middle = dict(case, quality=(case["quality"] + case["quality_high"]) // 2, sigma=(case["sigma"] + case["sigma_high"]) / 2)
    middle.update(quality_high=middle["quality"], sigma_high=middle["sigma"])
    device = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")
    h, w = min(case["height"], 512), min(case["width"], 512)
    sample = _files(middle, 1, device, images=1, height=h, width=w)[0]
    sample_units = -(-w // (8 * hs)) * -(-h // (8 * vs)) * (1 if ncomp == 1 else hs * vs + 2)
    d = _DENOMINATOR.get(case["output"], 1)
    samples = -(-case["width"] // d) * -(-case["height"] // d) * ncomp * case["images"]
    if case["output"] == "planar":
        chroma = -(-case["width"] // hs) * -(-case["height"] // vs)
        samples = (case["width"] * case["height"] + (ncomp - 1) * chroma) * case["images"]
    if case["output"] == "coefficients":
        samples = 0
    transform = 0 if case["output"] == "coefficients" else (16 * 36 + 64) / d ** 2
    scan_bytes = units * J.jpgd_parse(sample).scan_bytes / sample_units
    return {"bytes": scan_bytes + 128.0 * units + samples, "flops": units * transform + 3.0 * samples + units}


def tolerance(case):
    """Coefficients are whole numbers and must be the same.  Pixels are rounded from a 32-bit transform: two correct
    ones differ where the unrounded value lies within their rounding errors of a half.  Measured against the same
    transform in 64 bits, exact halves aside: at most 5e-5 of the samples of a full-size picture."""
    return "exact" if case["output"] == "coefficients" else {"rel": 0.0, "differ": 2e-4}
