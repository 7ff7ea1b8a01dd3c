"""GPU parity of the LZ4 decoders' steps: sequences at the edges of what a
window parses itself, chains over window edges, steps that end by bytes and by match count, matches
reading their own step, offsets past the LDS window."""
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


def _more(n):
    return b"\xff" * (n // 255) + bytes([n % 255])


def _seq(lits, match, off):
    n, m = len(lits), match - 4
    out = bytes([(min(n, 15) << 4) | (min(m, 15) if match else 0)])
    out += (_more(n - 15) if n >= 15 else b"") + lits
    if match:
        out += off.to_bytes(2, "little") + (_more(m - 15) if m >= 15 else b"")
    return out


def _block(rng, lit_choices, match_choices, off_choices, total):
    out, n = [], 0
    while n < total:
        k = int(rng.choice(lit_choices)) if n else max(1, int(rng.choice(lit_choices)))
        m = int(rng.choice(match_choices))
        off = max(1, min(n + k, 65535, int(rng.choice(off_choices))))
        out.append(_seq(rng.integers(0, 256, k, dtype=np.uint8).tobytes(), m, off))
        n += k + m
    last = rng.integers(0, 256, 7, dtype=np.uint8).tobytes()
    return b"".join(out) + _seq(last, 0, 0), n + 7


@pytest.mark.parametrize("lits,matches,offs", [
    ([0], [4], [1, 2, 3, 4, 5, 60, 300]),                          # as many matches as a window holds
    ([0, 1, 2, 3, 4, 7, 8, 13, 14], [4, 5, 8, 18, 19], [4, 17, 2000, 5000, 65535]),
    ([0, 14, 15, 16, 269, 270, 600], [4, 18, 19, 20, 272, 273, 274, 275], [1, 8, 273, 4096, 30000]),
    ([1], [273], [1, 7, 272, 273, 274]),                            # steps that end by bytes
    ([0, 1, 5], [511, 512, 513, 514, 515, 516, 1017, 1018, 1025, 1026], [1, 4, 7, 600]),  # matches made in pieces
    ([0, 14, 15, 268, 269, 270], [19, 273, 274, 528, 529, 1023, 1024, 1025, 1300], [1, 9, 1100, 20000]),
    ([0, 2000], [600, 1535, 1536, 2560, 9000], [1, 511, 512, 513, 6000]),
])
def test_steps(dev, lits, matches, offs):
    rng = np.random.default_rng(len(lits) * 100 + len(matches))
    blobs, sizes = zip(*[_block(rng, lits, matches, offs, total) for total in (1, 500, 2560, 9000, 31000, 100000)])
    ch = workloads._pack([oracle.LZ4] * len(blobs), list(blobs), list(sizes))
    assert (assert_parity(oracle.LZ4, ch, dev) == 0).all()                      # a team a block
    assert (assert_parity(oracle.LZ4, ch, dev, waves_per_block=1) == 0).all()   # a wave a block
    # The same blocks with an output range that ends inside a step, cut input
    # and an offset that reaches before the chunk.
    bad, caps = [], []
    for b, n in zip(blobs, sizes):
        for cap in (n - 1, n + 1, n // 2):
            bad.append(b)
            caps.append(cap)
        bad.append(b[: 2 * len(b) // 3])
        caps.append(n)
        bad.append(_seq(b"ab", 9, 3) + b)
        caps.append(n + 11)
    ch = workloads._pack([oracle.LZ4] * len(bad), bad, caps)
    st = assert_parity(oracle.LZ4, ch, dev)
    assert (st != 0).all() and (assert_parity(oracle.LZ4, ch, dev, waves_per_block=1) == st).all()
