"""The launch that a call selects by itself is not much slower than one that its
options select, on inputs that it is not at its best with.  Times are the best of
several, taken in turn; the bounds leave a wide margin."""
import zlib

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03760_amd as codag
    codag.lib()
    return torch.device("cuda:0")


def _best(calls):
    import torch
    best = [float("inf")] * len(calls)
    for _ in range(7):
        for i, call in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            call()
            a.record()
            for _ in range(4):
                call()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b))
    return best


def _ratio(dev, codec, blobs, sizes, **other):
    """Time by default over time with the options `other`."""
    import torch
    import paper_2307_03760_amd as codag
    comp = torch.from_numpy(np.frombuffer(b"".join(blobs) + b"\0" * 64, np.uint8).copy()).to(dev)
    co, oo = (torch.from_numpy(np.concatenate([[0], np.cumsum(k)]).astype(np.int64)).to(dev)
              for k in ([len(b) for b in blobs], sizes))
    out = torch.empty(int(sum(sizes)), dtype=torch.uint8, device=dev)
    st = torch.zeros(len(blobs), dtype=torch.int32, device=dev)
    own, theirs = _best([lambda: codag.decompress(codec, comp, co, out, oo, status=st),
                         lambda: codag.decompress(codec, comp, co, out, oo, status=st, **other)])
    assert not st.any()
    return own / theirs


def _deflate(data):
    c = zlib.compressobj(6, zlib.DEFLATED, -15)
    return c.compress(data) + c.flush()


def _text(size, seed):
    return workloads.zipf_text(size, np.random.default_rng(seed), workloads._vocab(0))


def test_deflate_chunks_of_uneven_sizes(dev):
    """One chunk in four long, in no order: workgroups of several waves would keep
    the LDS of those that are done."""
    data = [_text(65536 if k % 4 == 0 else 4096, k) for k in range(64)]
    blobs, sizes = [_deflate(d) for d in data], [len(d) for d in data]
    pick = np.random.default_rng(1).integers(0, 64, 10240)
    assert _ratio(dev, oracle.DEFLATE, [blobs[k] for k in pick], [sizes[k] for k in pick], waves_per_block=1) < 1.15


@pytest.mark.parametrize("n", [64, 600])
def test_deflate_short_blocks(dev, n):
    """Blocks of some 50 to 100 bytes, against the window-by-window decoder."""
    blobs = []
    for k in range(16):
        c, data = zlib.compressobj(6, zlib.DEFLATED, -15), _text(16384, k)
        blobs.append(b"".join(c.compress(data[i:i + 100]) + c.flush(zlib.Z_SYNC_FLUSH) for i in range(0, 16384, 100))
                     + c.flush())
    pick = np.random.default_rng(2).integers(0, 16, n)
    assert _ratio(dev, oracle.DEFLATE, [blobs[k] for k in pick], [16384] * n, variant=2) < 1.5


def _lz4_long_runs(seed):
    """Literal runs of 300 to 2,000 bytes between short matches."""
    rng, out, n = np.random.default_rng(seed), [], 0
    while n < 64000:
        k, m = int(rng.integers(300, 2001)), int(rng.integers(4, 18))
        off = int(rng.integers(1, min(n + k, 60000) + 1))
        out.append(bytes([0xF0 | (m - 4)]) + b"\xff" * ((k - 15) // 255) + bytes([(k - 15) % 255]) + rng.bytes(k)
                   + off.to_bytes(2, "little"))
        n += k + m
    return b"".join(out) + b"\x50tails", n + 5


@pytest.mark.parametrize("n", [64, 300, 1024])
def test_lz4_long_literal_runs(dev, n):
    blobs, sizes = zip(*[_lz4_long_runs(k) for k in range(16)])
    pick = np.random.default_rng(3).integers(0, 16, n)
    assert _ratio(dev, oracle.LZ4, [blobs[k] for k in pick], [sizes[k] for k in pick], waves_per_block=1) < 2


@pytest.mark.parametrize("size", [200, 4096])
def test_lz4_small_blocks(dev, size):
    blobs = [workloads.lz4_block(_text(size, k)) for k in range(16)]
    pick = np.random.default_rng(4).integers(0, 16, 1024)
    assert _ratio(dev, oracle.LZ4, [blobs[k] for k in pick], [size] * 1024, waves_per_block=1) < 2


def test_deflate_chunks_that_repeat(dev):
    """Every fourth chunk long: workgroups of one chunk, dealt to the XCDs in turn,
    would leave most of the XCDs idle."""
    data = [_text(65536 if k % 4 == 0 else 4096, k) for k in range(64)]
    blobs, sizes = [_deflate(d) for d in data], [len(d) for d in data]
    assert _ratio(dev, oracle.DEFLATE, blobs * 160, sizes * 160, waves_per_block=4) < 0.8
