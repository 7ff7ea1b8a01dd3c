"""GPU parity of byte RLE by one workgroup per chunk: groups across window edges
(4,096 byte positions, 2,048 in launches of more than 512 chunks), chains of the shortest and longest groups, ends and
errors anywhere; the one-wave decoder gives the same."""
import numpy as np
import pytest

import oracle
import workloads
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


def _stream(rng, groups):
    """groups: positive = a run of that length (3..130), negative = that many literals."""
    out = []
    for g in groups:
        out.append(bytes([g - 3, int(rng.integers(256))]) if g > 0 else bytes([256 + g]) + rng.bytes(-g))
    return b"".join(out), int(np.abs(groups).sum()) if len(groups) else 0


def _check(dev, blobs, sizes):
    ch = workloads._pack([oracle.BYTE_RLE] * len(blobs), blobs, sizes)
    st = assert_parity(oracle.BYTE_RLE, ch, dev)
    assert (assert_parity(oracle.BYTE_RLE, ch, dev, group_parallel=1) == st).all()
    k = 513 // len(blobs) + 1
    ch = workloads._pack([oracle.BYTE_RLE] * (len(blobs) * k), blobs * k, sizes * k)
    assert (assert_parity(oracle.BYTE_RLE, ch, dev, guards=False) == np.tile(st, k)).all()
    return st


@pytest.mark.parametrize("kinds", [[3], [130], [-1], [-128], [3, -1], [130, -128], list(range(3, 20)) + list(range(-20, 0))])
def test_group_shapes(dev, kinds):
    rng = np.random.default_rng(3)
    blobs, sizes = zip(*[_stream(rng, rng.choice(kinds, n)) for n in (0, 1, 7, 8, 9, 300, 1023, 1024, 1025, 5000)])
    assert (_check(dev, list(blobs), list(sizes)) == 0).all()


def test_ends_and_errors(dev):
    rng = np.random.default_rng(4)
    blobs, sizes = [], []
    for _ in range(6):
        b, n = _stream(rng, rng.choice([3, 10, 130, -1, -5, -128], 200))
        for cut in (1, 2, len(b) - 1, len(b) // 2, 2047, 2048, 2049):
            blobs.append(b[:cut])
            sizes.append(n)
        for cap in (0, 1, n - 1, n + 1, n // 2, n // 3):
            blobs.append(b)
            sizes.append(cap)
        blobs.append(b + b"\x00")
        sizes.append(n)
        for _ in range(10):
            m = bytearray(b)
            m[int(rng.integers(0, len(m)))] ^= 1 << int(rng.integers(0, 8))
            blobs.append(bytes(m))
            sizes.append(n)
    assert (_check(dev, blobs, sizes) != 0).sum() > 60
