"""GPU parity of RLE v2 by a workgroup per chunk: chunks shorter than its ranges,
around the length that one wave decodes alone, and long; runs over range cuts;
errors in every range; the one-wave decoder gives the same."""
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


@pytest.mark.parametrize("eb,uns", [(8, False), (8, True), (4, True), (2, False), (1, False)])
def test_lengths_and_errors(dev, eb, uns):
    rng = np.random.default_rng(eb + 16 * uns)
    blobs, sizes = [], []
    for n in (1, 2, 7, 8, 9, 100, 1535, 1536, 1537, 1600, 5000, 33000):
        src = workloads.rle_v2_workload(seed=n, n_values=n, chunk_values=n)
        blobs.append(src.comp[:int(src.chunk_offsets[1])].tobytes())
        sizes.append(eb * (int(src.out_offsets[1]) // 8))
    kw = {"elem_bytes": eb, "unsigned_values": uns}
    ch = workloads._pack([oracle.RLE_V2] * len(blobs), blobs, sizes)
    assert (assert_parity(oracle.RLE_V2, ch, dev, **kw) == 0).all()
    bad, caps = [], []
    for b, n in zip(blobs, sizes):
        for cap in (n - eb, n + eb, n // eb // 2 * eb):
            bad.append(b)
            caps.append(cap)
        bad.append(b + b"\x00")
        caps.append(n)
        for _ in range(12):
            m = bytearray(b)
            m[int(rng.integers(0, len(m)))] ^= 1 << int(rng.integers(0, 8))
            bad.append(bytes(m[: len(m) - int(rng.integers(0, 2))]))
            caps.append(n)
    ch = workloads._pack([oracle.RLE_V2] * len(bad), bad, caps)
    st = assert_parity(oracle.RLE_V2, ch, dev, **kw)
    assert (st != 0).sum() > 30
    assert (assert_parity(oracle.RLE_V2, ch, dev, group_parallel=1, **kw) == st).all()
