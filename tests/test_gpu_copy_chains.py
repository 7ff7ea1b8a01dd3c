"""GPU parity of a team's copies where steps hold as many as the queue takes and
every one reads the one before: hops over hops in all waves at once."""
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


@pytest.mark.parametrize("waves16", [True, False])
def test_deflate_chains(dev, waves16):
    """Copies of three bytes in 12 bits: 2,560 (or 1,280) of them fill the queue to its last entry."""
    rng = np.random.default_rng(11)
    blobs, sizes = [], []
    for dists in ([3], [4], [3, 4], [3, 6, 9, 12], [300], [3, 300]):
        w = BitWriter()
        w.put(1, 1)
        w.put(1, 2)
        n = max(dists)
        for v in rng.integers(0, 144, n):
            fixed_litlen(w, int(v))
        for d in rng.choice(dists, 7000):
            fixed_copy(w, 3, int(d))
            n += 3
        fixed_litlen(w, 256)
        blobs.append(w.getvalue())
        sizes.append(n)
    k = 1 if waves16 else 300 // len(blobs)
    ch = workloads._pack([oracle.DEFLATE] * (len(blobs) * k), blobs * k, sizes * k)
    assert (assert_parity(oracle.DEFLATE, ch, dev, guards=waves16) == 0).all()


def test_lz4_chains(dev):
    """Sequences of three bytes from every phase of the 3,072-position window: up
    to 1,024 matches a step."""
    rng = np.random.default_rng(12)
    blobs, sizes = [], []
    for first in range(1, 14):
        for offs in ([4], [4, 8], [1, 4]):
            lits = rng.integers(0, 256, first, dtype=np.uint8).tobytes()
            out, n = [bytes([first << 4]) + lits + (1).to_bytes(2, "little")], first + 4
            for o in rng.choice(offs, 4000):
                out.append(b"\0" + int(min(o, n)).to_bytes(2, "little"))
                n += 4
            out.append(bytes([5 << 4]) + b"tails")
            blobs.append(b"".join(out))
            sizes.append(n + 5)
    ch = workloads._pack([oracle.LZ4] * len(blobs), blobs, sizes)
    assert (assert_parity(oracle.LZ4, ch, dev) == 0).all()
