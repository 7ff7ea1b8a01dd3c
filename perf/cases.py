"""The work that programs give this library, as cases that can be timed.

Each case is one pass through a public entry point -- ``decompress``, a
``Plan``'s batched ``decompress`` or ``orc_decompress_stream`` -- on seeded
synthetic chunks: the compressed bytes are on the GPU, the output buffer is
allocated, and the pass enqueues the decode.  Sizes follow the repository's
workloads (64 and 2,048 RLE v1 chunks of 16,384 values, 1,024 RLE v2 chunks of
32,768 values, 16,384 Deflate chunks of 64 KiB, log-normal batches) and what
ORC writers produce by default (row groups of 10,000 values, 64 and 256 KiB
compression blocks).  Large cases repeat a set of distinct chunks; every chunk
has its own place in the input and in the output.

All outputs are bytes and statuses, so there is nothing to compute in 64 bits.
"""
import math
import zlib
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2307_03760_amd as codag

MIB = 1 << 20


def listed():
    return [
        # One ORC row group of an integer column: the smallest call a reader makes.
        {"name": "rle_v2_row_group", "path": "rle_v2", "chunks": 1, "values": 10000, "elem": 8, "signed": True},
        # The repository's RLE v1 workload: few chunks, group-parallel decode.
        {"name": "rle_v1_64", "path": "rle_v1", "chunks": 64, "values": 16384, "elem": 8, "signed": True},
        # A table scan's worth of RLE v1 chunks, one wave each, the last ones ragged.
        {"name": "rle_v1_2043", "path": "rle_v1", "chunks": 2043, "values": 16384, "elem": 8, "signed": True},
        # The repository's RLE v2 workload (its headline).
        {"name": "rle_v2_1024", "path": "rle_v2", "chunks": 1024, "values": 32768, "elem": 8, "signed": True},
        # String lengths of 300 row groups, as ORC stores them: unsigned, into 32-bit values.
        {"name": "rle_v2_lengths_u32", "path": "rle_v2", "chunks": 300, "values": 10000, "elem": 4, "signed": False},
        # Byte columns (tinyint, bitmaps) of some hundred stripes' row groups.
        {"name": "byte_rle_400", "path": "byte_rle", "chunks": 400, "values": 50000, "elem": 1, "signed": True},
        # The repository's Deflate workload: 1 GiB in 64 KiB chunks.
        {"name": "deflate_16384", "path": "deflate", "chunks": 16384, "size": 65536, "level": 9},
        # A small read: a few dozen pages of odd size.
        {"name": "deflate_48_odd", "path": "deflate", "chunks": 48, "size": 60001, "level": 6},
        # One compressed ORC stream, ZLIB, the default 256 KiB block.
        {"name": "orc_zlib_12m", "path": "orc_zlib", "bytes": 12 * MIB + 4321, "block": 262144, "level": 6},
        # LZ4 blocks of a large file.
        {"name": "lz4_4096", "path": "lz4", "chunks": 4096, "size": 65536},
        # One compressed ORC stream, LZ4, 64 KiB blocks.
        {"name": "orc_lz4_6m", "path": "orc_lz4", "bytes": 6 * MIB + 777, "block": 65536, "level": 0},
        # A batch of mixed codecs and uneven sizes in one launch, queued by the learned order.
        {"name": "batch_learned_2000", "path": "batch", "chunks": 2000, "order": "learned", "median": 65536},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["rle_v1", "rle_v2", "byte_rle", "deflate", "deflate", "lz4", "orc_zlib", "orc_lz4", "batch"])
    if path in ("rle_v1", "rle_v2"):
        chunks = _log(rng, 1, 4096)
        values = _log(rng, 500, min(60000, (1 << 25) // chunks))
        elem, signed = rng.choice([(8, True), (8, True), (4, False), (4, True), (2, True)])
        return {"path": path, "chunks": chunks, "values": values, "elem": elem, "signed": signed}
    if path == "byte_rle":
        chunks = _log(rng, 1, 4096)
        return {"path": path, "chunks": chunks, "values": _log(rng, 500, min(200000, (1 << 26) // chunks)), "elem": 1, "signed": True}
    if path == "deflate":
        chunks = _log(rng, 1, 8192)
        return {"path": path, "chunks": chunks, "size": _log(rng, 4096, min(262144, 512 * MIB // chunks)), "level": rng.choice([6, 9])}
    if path == "lz4":
        chunks = _log(rng, 1, 4096)
        return {"path": path, "chunks": chunks, "size": _log(rng, 4096, min(131072, 256 * MIB // chunks))}
    if path in ("orc_zlib", "orc_lz4"):
        return {"path": path, "bytes": _log(rng, 20000, 24 * MIB), "block": rng.choice([32768, 65536, 262144]), "level": 6 if path == "orc_zlib" else 0}
    return {"path": path, "chunks": _log(rng, 200, 2500), "order": rng.choice(["index", "learned"]), "median": rng.choice([16384, 65536])}


# ---------------------------------------------------------------------------
# Values and their encodings
# ---------------------------------------------------------------------------

def _varints(z):
    """Base-128 varints of unsigned 64-bit values: (all bytes, end of each)."""
    z = np.asarray(z, dtype=np.uint64)
    shifted = z[:, None] >> (np.uint64(7) * np.arange(10, dtype=np.uint64))[None, :]
    more = np.concatenate([shifted[:, 1:] != 0, np.zeros((z.size, 1), bool)], axis=1)
    b = (shifted & np.uint64(0x7F)).astype(np.uint8) | (more.astype(np.uint8) << 7)
    n = 1 + more.sum(axis=1)
    return b[np.arange(10)[None, :] < n[:, None]].tobytes(), np.cumsum(n)


def _zigzag(v):
    v = np.asarray(v, dtype=np.int64)
    return (v.astype(np.uint64) << np.uint64(1)) ^ (v >> np.int64(63)).astype(np.uint64)


def _code(v, signed):
    return _zigzag(v) if signed else np.asarray(v, dtype=np.int64).astype(np.uint64)


def _span(elem, signed):
    """Bits of the magnitudes that a column of this type holds."""
    return {8: 40, 4: 20 if not signed else 30, 2: 14}[elem]


def _rle_v1_chunk(rng, n, elem, signed):
    """Runs of 3..130 values (delta -128..127) and literal lists of 1..128, alternating."""
    hi = 1 << _span(elem, signed)
    lo = -hi if signed else 0
    out, left, run = [], n, True
    lits, at = _varints(_code(rng.integers(lo, hi, n), signed))
    at = np.concatenate([[0], at])
    used = 0
    while left:
        if run and left >= 3:
            k = min(left, int(rng.integers(3, 131)))
            delta = int(rng.integers(-128, 128)) if signed else int(rng.integers(0, 4))
            out.append(bytes([k - 3, delta & 255]) + _varints(_code([int(rng.integers(lo, hi))], signed))[0])
        else:
            k = min(left, int(rng.integers(1, 129)))
            out.append(bytes([256 - k]) + lits[at[used]:at[used + k]])
            used += k
        left -= k
        run = not run
    return b"".join(out)


_WIDTHS = list(range(1, 25)) + [26, 28, 30, 32, 40, 48, 56, 64]


def _width(bits):
    return next(w for w in _WIDTHS if w >= bits)


def _packed(v, w):
    v = np.asarray(v, dtype=np.uint64)
    bits = (v[:, None] >> np.arange(w - 1, -1, -1, dtype=np.uint64)[None, :]) & np.uint64(1)
    return np.packbits(bits.astype(np.uint8).reshape(-1)).tobytes()


def _head(kind, w, n):
    return bytes([(kind << 6) | (_WIDTHS.index(w) << 1) | ((n - 1) >> 8), (n - 1) & 255])


def _rle_v2_chunk(rng, n, elem, signed):
    """About a quarter of the values each as SHORT_REPEAT (3..10), DIRECT, DELTA
    and PATCHED_BASE runs of up to 512."""
    top = 64 if elem == 8 else _span(elem, signed)
    out, left = [], n
    odds = 1 - 3 * 6.5 / 512
    while left:
        if left < 3 or (left >= 3 and rng.random() < odds):
            k = min(left, int(rng.integers(3, 11)))
            if k >= 3:
                nb = int(rng.integers(1, min(8, max(1, (top + 7) // 8)) + 1))
                out.append(bytes([((nb - 1) << 3) | (k - 3)]) + rng.bytes(nb))
            else:
                out.append(_head(1, 8, k) + rng.bytes(k))
            left -= k
            continue
        k, kind = min(left, 512), int(rng.integers(3))
        if kind == 0:
            w = _width(int(rng.integers(1, top + 1)))
            out.append(_head(1, w, k) + rng.bytes((k * w + 7) // 8))
        elif kind == 1 and k >= 3:
            step, w = rng.integers(1, 1001, k - 2), 10
            base = int(rng.integers(0, 1 << min(40, top)))
            out.append(_head(3, w, k) + _varints(_code([base], signed))[0] + _varints(_zigzag([int(step[0])]))[0] + _packed(step, w))
        else:
            # Values below 2^12, 2% outliers patched above them (gap 8 bits, patch 24 or 8 bits).
            pw = 24 if elem == 8 else 8
            at = np.unique(rng.integers(0, k, max(1, min(20, k // 50))))
            at = at[np.diff(np.concatenate([[0], at])) < 256]
            gaps = np.diff(np.concatenate([[0], at]))
            keep = np.cumsum(gaps) < k
            entries = (gaps[keep].astype(np.uint64) << np.uint64(pw)) | rng.integers(1, 1 << pw, int(keep.sum())).astype(np.uint64)
            h = _head(2, 12, k)
            out.append(h + bytes([(1 << 5) | _WIDTHS.index(pw), (7 << 5) | entries.size]) + bytes([0, int(rng.integers(0, 100))]) +
                       _packed(rng.integers(0, 4096, k), 12) + _packed(entries, _width(8 + pw)))
        left -= k
    return b"".join(out)


def _byte_rle_chunk(rng, n):
    """Byte runs of 3..130 and literal lists of 1..128 bytes, alternating."""
    out, left, run = [], n, True
    while left:
        if run and left >= 3:
            k = min(left, int(rng.integers(3, 131)))
            out.append(bytes([k - 3, int(rng.integers(256))]))
        else:
            k = min(left, int(rng.integers(1, 129)))
            out.append(bytes([256 - k]) + rng.bytes(k))
        left -= k
        run = not run
    return b"".join(out)


# ---------------------------------------------------------------------------
# Bytes for Deflate and LZ4
# ---------------------------------------------------------------------------

class _Text:
    """Zipf(1.1) text over 4,096 random lowercase words."""

    def __init__(self, rng):
        n = rng.integers(3, 11, 4096)
        self.words = [bytes(rng.integers(97, 123, int(k), dtype=np.uint8)) + b" " for k in n]
        p = np.arange(1, 4097, dtype=np.float64) ** -1.1
        self.cdf = np.cumsum(p / p.sum())

    def take(self, rng, size):
        ids = np.minimum(np.searchsorted(self.cdf, rng.random(size // 4 + 16)), 4095)
        return b"".join([self.words[i] for i in ids])[:size]


def _content(rng, text, kind, size):
    if kind == "text":
        return text.take(rng, size)
    if kind == "random":
        return rng.bytes(size)
    distinct = rng.integers(-(1 << 31), 1 << 31, 64).astype("<i4")
    n = size // 4 + 1
    if kind == "int32":
        return distinct[rng.integers(0, 64, n)].tobytes()[:size]
    length = np.floor(np.exp(rng.uniform(math.log(2), math.log(201), n // 2 + 2))).astype(np.int64)
    return np.repeat(distinct[rng.integers(0, 64, length.size)], length)[:n].tobytes().ljust(size, b"\0")[:size]


def _kinds(rng, n):
    """Half text, three tenths columns (a third of them runs), a fifth random, in seeded order."""
    few = ["text", "int32", "text", "random", "text", "int32_runs", "text", "int32", "text", "random"]
    return [few[i % 10] for i in rng.permutation(10 * ((n + 9) // 10))[:n]]


def _deflate(data, level, fixed=False):
    c = zlib.compressobj(level, zlib.DEFLATED, -15, 8, zlib.Z_FIXED if fixed else zlib.Z_DEFAULT_STRATEGY)
    return c.compress(data) + c.flush()


def _lz4(data):
    """A greedy LZ4 block: matches found through a table of the next four bytes."""
    n, out, table = len(data), [], {}
    anchor = i = 0

    def sequence(lit, match, off):
        m = match - 4
        head = bytes([(min(len(lit), 15) << 4) | (min(m, 15) if off else 0)])
        for v in (len(lit),):
            if v >= 15:
                head += b"\xff" * ((v - 15) // 255) + bytes([(v - 15) % 255])
        tail = b""
        if off:
            tail = off.to_bytes(2, "little")
            if m >= 15:
                tail += b"\xff" * ((m - 15) // 255) + bytes([(m - 15) % 255])
        out.append(head + lit + tail)

    skip = 0
    while i < n - 12:
        key = data[i:i + 4]
        j = table.get(key)
        table[key] = i
        if j is None or i - j > 65535:
            skip += 1
            i += 1 + (skip >> 6)
            continue
        skip, m, most = 0, 4, n - 5 - i
        while m + 16 <= most and data[j + m:j + m + 16] == data[i + m:i + m + 16]:
            m += 16
        while m < most and data[j + m] == data[i + m]:
            m += 1
        sequence(data[anchor:i], m, i - j)
        i += m
        anchor = i
    sequence(data[anchor:], 4, 0)
    return b"".join(out)


def _pack_map(fn, items):
    with ThreadPoolExecutor(8) as ex:
        return list(ex.map(fn, items))


# ---------------------------------------------------------------------------
# A case's chunks
# ---------------------------------------------------------------------------

# Distinct chunks of a case; larger ones repeat them.
_DISTINCT = {"rle_v1": 64, "rle_v2": 48, "byte_rle": 48, "deflate": 80, "lz4": 30}


def _batch_chunks(case, rng):
    """Codec and output bytes of each chunk of a batch: 40% RLE v1, 30% RLE v2,
    30% Deflate, log-normal sizes, grouped by codec so RLE outputs are aligned."""
    n = case["chunks"]
    codecs = np.sort(rng.choice([codag.RLE_V1, codag.RLE_V2, codag.DEFLATE], n, p=[0.4, 0.3, 0.3]))
    sizes = np.clip(np.exp(rng.normal(math.log(case["median"]), 1.0, n)), 4096, MIB).astype(np.int64)
    return codecs, np.where(codecs == codag.DEFLATE, sizes, sizes // 8 * 8)


def _encoded(case, seed):
    """(codec of each chunk, compressed chunks, output bytes of each)."""
    rng = np.random.default_rng([seed, 1])
    shape = np.random.default_rng(1)  # sizes and content classes belong to the case, not to its inputs
    path = case["path"]
    if path in ("rle_v1", "rle_v2", "byte_rle"):
        n, d = case["chunks"], min(case["chunks"], _DISTINCT[path])
        # Chunk sizes vary by a few per cent, as row groups cut at a byte or row limit do.
        count = [case["values"] - (int(shape.integers(0, case["values"] // 32 + 1)) if k % 3 == 2 else 0) for k in range(d)]
        if path == "byte_rle":
            blobs = [_byte_rle_chunk(rng, k) for k in count]
        else:
            enc = _rle_v1_chunk if path == "rle_v1" else _rle_v2_chunk
            blobs = [enc(rng, k, case["elem"], case["signed"]) for k in count]
        codec = {"rle_v1": codag.RLE_V1, "rle_v2": codag.RLE_V2, "byte_rle": codag.BYTE_RLE}[path]
        return np.full(n, codec), [blobs[i % d] for i in range(n)], [case["elem"] * count[i % d] for i in range(n)]
    text = _Text(rng)
    if path in ("deflate", "lz4"):
        n, d = case["chunks"], min(case["chunks"], _DISTINCT[path])
        sizes = [case["size"] if case["size"] % 4096 == 0 else case["size"] - int(shape.integers(0, case["size"] // 16 + 1)) for _ in range(d)]
        data = [_content(rng, text, k, s) for k, s in zip(_kinds(shape, d), sizes)]
        if path == "lz4":
            blobs = [_lz4(x) for x in data]
        else:
            fixed = shape.random(d) < 1 / 3 if case["level"] == 9 else np.zeros(d, bool)
            blobs = _pack_map(lambda a: _deflate(a[0], case["level"], bool(a[1])), list(zip(data, fixed)))
        codec = codag.DEFLATE if path == "deflate" else codag.LZ4
        return np.full(n, codec), [blobs[i % d] for i in range(n)], [sizes[i % d] for i in range(n)]
    if path in ("orc_zlib", "orc_lz4"):
        # A stream of column data: dictionary text and integer columns, a little of it incompressible.
        block, total = case["block"], case["bytes"]
        n = -(-total // block)
        d = min(n, max(2, 3 * MIB // block))
        kinds = [["text", "int32", "text", "int32_runs", "text", "int32", "text", "random"][i % 8] for i in range(d)]
        data = [_content(rng, text, k, block) for k in kinds]
        sizes = [min(block, total - i * block) for i in range(n)]
        pack = (lambda x: _deflate(x, case["level"])) if path == "orc_zlib" else _lz4
        whole = _pack_map(pack, data)
        blobs = [whole[i % d] if s == block else pack(data[i % d][:s]) for i, s in enumerate(sizes)]
        framed = []
        for i, b in enumerate(blobs):
            raw = len(b) >= sizes[i]
            b = data[i % d][:sizes[i]] if raw else b
            framed.append(((len(b) << 1) | int(raw)).to_bytes(3, "little") + b)
        return np.full(n, 0), framed, sizes
    codecs, sizes = _batch_chunks(case, shape)
    # One long chunk of each kind, cut to size by encoding prefixes, would cost
    # as much as encoding each; instead each chunk takes the size of one of a
    # set of distinct chunks nearest to its own.
    blobs, out = [], []
    for codec in (codag.RLE_V1, codag.RLE_V2, codag.DEFLATE):
        want = sizes[codecs == codec]
        if not want.size:
            continue
        have = np.unique(np.quantile(want, np.linspace(0, 1, 40)).astype(np.int64) // 8 * 8 + (3 if codec == codag.DEFLATE else 0))
        kinds = _kinds(shape, have.size)
        if codec == codag.DEFLATE:
            fixed = shape.random(have.size) < 1 / 3
            enc = _pack_map(lambda a: _deflate(a[0], 9, bool(a[1])), [(_content(rng, text, k, int(s)), f) for k, s, f in zip(kinds, have, fixed)])
        else:
            make = _rle_v1_chunk if codec == codag.RLE_V1 else _rle_v2_chunk
            enc = [make(rng, int(s) // 8, 8, True) for s in have]
        at = np.abs(want[:, None] - have[None, :]).argmin(axis=1)
        blobs += [enc[i] for i in at]
        out += [int(have[i]) for i in at]
    return codecs, blobs, out


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(np.asarray(sizes, dtype=np.int64))])


def prepare(case, seed):
    codecs, blobs, sizes = _encoded(case, seed)
    comp = torch.from_numpy(np.frombuffer(b"".join(blobs), dtype=np.uint8).copy()).cuda()
    out_off = _offsets(sizes)
    s = {"path": case["path"], "comp": comp, "out": torch.zeros(int(out_off[-1]), dtype=torch.uint8, device="cuda")}
    if case["path"] in ("orc_zlib", "orc_lz4"):
        s["codec"] = codag.DEFLATE if case["path"] == "orc_zlib" else codag.LZ4
        s["block"] = case["block"]
        s["len"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        return s
    s["off"] = torch.from_numpy(_offsets([len(b) for b in blobs])).cuda()
    s["out_off"] = torch.from_numpy(out_off).cuda()
    s["status"] = torch.zeros(len(blobs), dtype=torch.int32, device="cuda")
    if case["path"] == "batch":
        s["codecs"] = torch.from_numpy(codecs.astype(np.uint8)).cuda()
        learned = case["order"] == "learned"
        s["plan"] = codag.Plan(order=codag.ORDER_LEARNED if learned else codag.ORDER_INDEX, use_graph=True)
        if learned:  # fitted once, on what the chunks' decode took
            ticks = torch.zeros(len(blobs), dtype=torch.int64, device="cuda")
            s["plan"].decompress(s["codecs"], comp, s["off"], s["out"], s["out_off"], chunk_ticks=ticks)
            feat = s["plan"].features(s["codecs"], comp, s["off"], s["out_off"])
            s["plan"].train(feat, torch.log2(ticks.float() + 1), steps=150, lr=2e-3, seed=1 + seed % 1000)
        return s
    s["codec"] = int(codecs[0])
    s["elem"] = case.get("elem", 8)
    s["unsigned"] = not case.get("signed", True)
    return s


def run(s):
    if s["path"] in ("orc_zlib", "orc_lz4"):
        codag.orc_decompress_stream(s["codec"], s["comp"], s["block"], s["out"], s["len"], s["status"])
        return [s["out"], s["len"], s["status"]]
    if s["path"] == "batch":
        s["plan"].decompress(s["codecs"], s["comp"], s["off"], s["out"], s["out_off"], status=s["status"])
    elif s["path"] in ("rle_v1", "rle_v2"):
        codag.decompress(s["codec"], s["comp"], s["off"], s["out"], s["out_off"], status=s["status"],
                         elem_bytes=s["elem"], unsigned_values=s["unsigned"])
    else:
        codag.decompress(s["codec"], s["comp"], s["off"], s["out"], s["out_off"], status=s["status"])
    return [s["out"], s["status"]]


def work(case):
    """Every compressed byte read once, every output byte written once, and the
    offsets.  Decoding has no floating-point work."""
    _, blobs, sizes = _encoded(case, 0)
    return {"bytes": sum(map(len, blobs)) + sum(sizes) + 16 * len(blobs), "flops": 0}


def exact(case, seed):
    return None  # bytes and whole numbers
