"""GPU parity of the lane-parallel Deflate decoder at its own edges: rounds of
256 bits a lane (one wave, or a team of 8 or 16 waves), 64-bit segments, steps bounded by output and copy count, codes
that never fall back onto the track, errors inside a round."""
import zlib

import numpy as np
import pytest

import oracle
import workloads
from deflate_bits import BitWriter, fixed_copy, fixed_litlen
from gpu_util import assert_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03760_amd as codag
    codag.lib()
    return torch.device("cuda:0")


def _z(data, level=6, strategy=zlib.Z_DEFAULT_STRATEGY):
    c = zlib.compressobj(level, zlib.DEFLATED, -15, 8, strategy)
    return c.compress(data) + c.flush()


def _check(dev, blobs, sizes):
    """By teams of 16 waves, of 8 (more than 256 chunks) and by one wave a chunk."""
    ch = workloads._pack([oracle.DEFLATE] * len(blobs), blobs, sizes)
    st = assert_parity(oracle.DEFLATE, ch, dev)
    assert (assert_parity(oracle.DEFLATE, ch, dev, waves_per_block=1) == st).all()
    k = 257 // len(blobs) + 1
    if sum(sizes) * k < 1 << 28 and len(blobs) * k <= 512:
        ch = workloads._pack([oracle.DEFLATE] * (len(blobs) * k), blobs * k, sizes * k)
        assert (assert_parity(oracle.DEFLATE, ch, dev, guards=False) == np.tile(st, k)).all()
    return st


def _literals(bits_wanted):
    """A fixed block of 8-bit literals whose end-of-block code starts at the given bit."""
    w = BitWriter()
    w.put(1, 1)
    w.put(1, 2)
    n = 0
    nine = (bits_wanted - 3) % 8  # a nine-bit literal moves the block's end by one bit
    for _ in range(nine):
        fixed_litlen(w, 200)
        n += 1
    while len(w.bits) + 8 <= bits_wanted:
        fixed_litlen(w, 65 + n % 26)
        n += 1
    assert len(w.bits) == bits_wanted
    fixed_litlen(w, 256)
    return w.getvalue(), n


@pytest.mark.parametrize("around", [64, 256, 512, 64 * 256, 64 * 256 + 64, 512 * 256, 1024 * 256])
def test_block_ends_at_segment_lane_and_round_edges(dev, around):
    blobs, sizes = zip(*[_literals(b) for b in range(around - 9 + 80 * (around == 64), around + 10 + 80 * (around == 64))])
    assert (_check(dev, list(blobs), list(sizes)) == 0).all()


def test_codes_of_one_length_and_steps_of_every_shape(dev):
    rng = np.random.default_rng(5)
    alphabet = np.frombuffer(bytes(range(48, 112)), np.uint8)  # 64 symbols: six-bit codes
    datas = [alphabet[rng.integers(0, 64, n)].tobytes() for n in (50, 3000, 70001)]
    datas += [bytes(300000), b"ab" * 60000, bytes(range(256)) * 300]           # segments of many kilobytes
    noise = rng.integers(0, 256, 40000, dtype=np.uint8).tobytes()
    datas += [noise[:30000] + noise[:30000], (noise[:5000] + b"-") * 9]        # long far copies
    blobs, sizes = [], []
    for d in datas:
        for level, strategy in ((1, 0), (6, 0), (9, 0), (6, zlib.Z_HUFFMAN_ONLY), (6, zlib.Z_FIXED)):
            blobs.append(_z(d, level, strategy))
            sizes.append(len(d))
    assert (_check(dev, blobs, sizes) == 0).all()


def test_copies_of_every_length_and_distance_relation(dev):
    """Lengths 3..258 at distances below, at and above them and at the window's
    and the history's limits, one after another, many of them reading the
    copy before."""
    rng = np.random.default_rng(6)
    blobs, sizes = [], []
    for k in range(24):
        w = BitWriter()
        w.put(1, 1)
        w.put(1, 2)
        n = 0
        for _ in range(40 + 400 * (k % 5)):
            fixed_litlen(w, int(rng.integers(0, 256)))
            n += 1
        for _ in range(700):
            length = int(rng.choice([3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 34, 40, 63, 64, 65, 257, 258]))
            near = [1, 2, 3, 7, 8, 9, length - 1, length, length + 1, 300, 1535, 1536, 1537, 2560, 4095, 4096, 32768]
            d = max(1, min(n, int(rng.choice(near)) + int(rng.integers(0, 2))))
            fixed_copy(w, length, min(d, 32768))
            n += length
            if rng.random() < 0.3:
                fixed_litlen(w, int(rng.integers(0, 256)))
                n += 1
        fixed_litlen(w, 256)
        blobs.append(w.getvalue())
        sizes.append(n)
    assert (_check(dev, blobs, sizes) == 0).all()


def test_stored_blocks_and_history(dev):
    """Stored blocks of many lengths, with copies that read them and the text
    before them."""
    rng = np.random.default_rng(8)
    blobs, sizes = [], []
    for n in (1, 100, 4095, 4096, 4097, 5000, 20000, 65535):
        c = zlib.compressobj(6, zlib.DEFLATED, -15, 8)
        text = workloads.zipf_text(3000, rng, workloads._vocab(0))
        noise = rng.integers(0, 256, n, dtype=np.uint8).tobytes()
        data = [text, noise, text + noise[:300] + noise[-700:], noise[: n // 2], text]
        blobs.append(b"".join(c.compress(d) + c.flush(zlib.Z_FULL_FLUSH if i == 0 else zlib.Z_BLOCK)
                              for i, d in enumerate(data)) + c.flush())
        sizes.append(sum(map(len, data)))
    assert (_check(dev, blobs, sizes) == 0).all()


def test_errors_inside_a_round(dev):
    """A distance before the chunk, an output range that ends anywhere, input
    cut off anywhere and damaged bytes, in the middle of otherwise long
    rounds: the sequential decoder's status each time."""
    rng = np.random.default_rng(7)
    text = workloads.zipf_text(30000, rng, workloads._vocab(0))
    blobs, sizes = [], []
    for good in (_z(text), _z(text, 9, zlib.Z_FIXED)):
        for cap in (0, 1, 700, 1535, 1536, 1537, 9999, 29999, 30001):
            blobs.append(good)
            sizes.append(cap)
        for cut in (1, 40, 511, 2047, 2048, 2049, 5000):
            blobs.append(good[:cut])
            sizes.append(len(text))
        for _ in range(30):
            b = bytearray(good)
            b[int(rng.integers(60, len(b)))] ^= 1 << int(rng.integers(0, 8))
            blobs.append(bytes(b))
            sizes.append(len(text))
    for at in (1, 100, 1000, 3000):
        for over in (1, 2, 3000):
            w = BitWriter()
            w.put(1, 1)
            w.put(1, 2)
            for i in range(at):
                fixed_litlen(w, i % 200)
            fixed_copy(w, 5, at)
            fixed_copy(w, 9, at + 5 + over)
            for i in range(2000):
                fixed_litlen(w, i % 200)
            fixed_litlen(w, 256)
            blobs.append(w.getvalue())
            sizes.append(at + 14 + 2000)
    st = _check(dev, blobs, sizes)
    assert (st != 0).sum() > 40
