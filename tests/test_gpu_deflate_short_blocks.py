"""GPU parity of Deflate blocks around the lengths at which the decoder changes:
window by window, rounds of one wave, rounds of a team; alone in a chunk, after
blocks of other lengths, with flushes in between, cut off and with too small an
output."""
import zlib

import numpy as np
import pytest

import oracle
import workloads
from deflate_bits import DIST_BASE, BitWriter, fixed_copy, fixed_litlen
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


def _stream(data, cuts, flushes, level=6, strategy=zlib.Z_DEFAULT_STRATEGY):
    c, out, a = zlib.compressobj(level, zlib.DEFLATED, -15, 8, strategy), [], 0
    for k, n in enumerate(cuts):
        out.append(c.compress(data[a:a + n]) + c.flush(flushes[k % len(flushes)]))
        a += n
    return b"".join(out) + c.compress(data[a:]) + c.flush()


@pytest.mark.parametrize("strategy", [zlib.Z_DEFAULT_STRATEGY, zlib.Z_FIXED, zlib.Z_HUFFMAN_ONLY])
def test_blocks_of_every_length(dev, strategy):
    rng = np.random.default_rng(21)
    vocab = workloads._vocab(0)
    blobs, sizes = [], []

    def add(data, cuts, flushes):
        blobs.append(_stream(data, cuts, flushes, 6, strategy))
        sizes.append(len(data))

    for n in list(range(0, 40)) + list(range(300, 1000, 20)) + [1500, 2500, 4000]:
        add(workloads.zipf_text(n, rng, vocab) if n else b"", [], [])
    kinds = [zlib.Z_SYNC_FLUSH, zlib.Z_PARTIAL_FLUSH, zlib.Z_BLOCK, zlib.Z_FULL_FLUSH]
    for per in (1, 10, 50, 200, 700, 900, 1200, 3000):
        data = workloads.zipf_text(12 * per + 7, rng, vocab)
        for f in kinds:
            add(data, [per] * 12, [f])
    for _ in range(12):  # short after long, long after short
        cuts = [int(c) for c in rng.choice([5, 60, 400, 1100, 5000, 30000], 8)]
        add(workloads.zipf_text(sum(cuts) + 100, rng, vocab), cuts, [kinds[int(rng.integers(4))], zlib.Z_SYNC_FLUSH])
    add(bytes(70000), [], [])
    for waves in (0, 1):  # teams where the launch is small, one wave a chunk
        ch = workloads._pack([oracle.DEFLATE] * len(blobs), blobs, sizes)
        assert (assert_parity(oracle.DEFLATE, ch, dev, waves_per_block=waves) == 0).all()
    bad, caps = [], []
    for b, n in zip(blobs[::3], sizes[::3]):
        bad += [b[:len(b) // 2], b[:-1], b, b]
        caps += [n, n, n // 2, n + 1]
    for waves in (0, 1):
        ch = workloads._pack([oracle.DEFLATE] * len(bad), bad, caps)
        assert_parity(oracle.DEFLATE, ch, dev, waves_per_block=waves)


@pytest.mark.parametrize("bits", [0, 9, 10])
def test_every_symbol_of_the_fixed_code(dev, bits):
    blobs, sizes = [], []
    for end in [None, 286, 287, (257, 30), (257, 31)]:  # a good block; symbols that may not appear
        for rounds in (1, 140):  # short, and long enough for the rounds
            w = BitWriter()
            w.put(1, 1)
            w.put(1, 2)
            n = 0
            for _ in range(rounds):
                for s in range(256):
                    fixed_litlen(w, s)
                n += 256
            for length in range(3, 259):
                fixed_copy(w, length, 1 + length % 256)
                n += length
            for d in DIST_BASE:
                if d <= n:
                    fixed_copy(w, 3, d)
                    n += 3
            if end is None:
                fixed_litlen(w, 256)
            elif isinstance(end, int):
                fixed_litlen(w, end)
            else:
                fixed_litlen(w, end[0])
                w.put_code(end[1], 5)
            w.put(0, 40)
            blobs.append(w.getvalue())
            sizes.append(n)
    ch = workloads._pack([oracle.DEFLATE] * len(blobs), blobs, sizes)
    st = assert_parity(oracle.DEFLATE, ch, dev, lit_table_bits=bits)
    assert (st[:2] == 0).all() and (st[2:] == oracle.E_CORRUPT).all()


@pytest.mark.parametrize("waves", [0, 1])
def test_short_blocks_of_much_output(dev, waves):
    """Few bits and many bytes: runs of integers, repeated bytes and phrases, alone
    and as blocks of a stream among short ones."""
    rng = np.random.default_rng(23)
    blobs, sizes = [], []
    for n in (100, 3000, 8192, 8193, 16000, 24000, 40000, 70000):
        runs = workloads.int32_column(n, rng, run_heavy=True)
        for data in (runs, bytes(n), (runs[:40] * (n // 40 + 1))[:n]):
            blobs.append(_stream(data, [], []))
            sizes.append(n)
            blobs.append(_stream(b"a few words" + data + data[:500], [11, n, 200, 200], [zlib.Z_BLOCK, zlib.Z_SYNC_FLUSH]))
            sizes.append(11 + n + min(n, 500))
            blobs.append(_stream(data * 3, [n, n, n], [zlib.Z_FULL_FLUSH]))
            sizes.append(3 * n)
    ch = workloads._pack([oracle.DEFLATE] * len(blobs), blobs, sizes)
    assert (assert_parity(oracle.DEFLATE, ch, dev, waves_per_block=waves) == 0).all()
