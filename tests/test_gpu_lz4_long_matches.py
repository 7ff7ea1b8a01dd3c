"""GPU parity of LZ4 matches far longer than the pieces they are made in, at
offsets below, at and above a piece's length; by a team and by one wave."""
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


@pytest.mark.parametrize("waves", [0, 1])
def test_long_matches(dev, waves):
    rng = np.random.default_rng(31)
    blobs, sizes = [], []
    for off in [1, 2, 3, 7, 8, 63, 64, 65, 251, 252, 253, 503, 504, 505, 511, 512, 513, 700, 1008, 1030, 2600]:
        for length in (1030, 5000, 40001):
            lits = rng.integers(0, 256, off + int(rng.integers(0, 9)), dtype=np.uint8).tobytes()
            out, n = b"", 0
            for k in range(2):
                head = bytes([(min(len(lits), 15) << 4) | 15]) + (_more(len(lits) - 15) if len(lits) >= 15 else b"")
                out += head + lits + off.to_bytes(2, "little") + _more(length - 19)
                n += len(lits) + length
                lits = lits[: 1 + k]
            blobs.append(out + bytes([6 << 4]) + b"ending")
            sizes.append(n + 6)
    ch = workloads._pack([oracle.LZ4] * len(blobs), blobs, sizes)
    assert (assert_parity(oracle.LZ4, ch, dev, waves_per_block=waves) == 0).all()
