"""Original (uncompressed) chunks of ORC streams come back whole, whatever their
length, in every launch that a stream's capacity selects: teams of 16 and of 8
waves a chunk and one wave a chunk."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BLOCK = 70000
LENGTHS = (list(range(1, 41)) + list(range(1020, 1028)) + list(range(8185, 8201)) + list(range(16380, 16401))
           + [32769, 32783] + list(range(65530, 65553)))


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03760_amd as codag
    codag.lib()
    return torch.device("cuda:0")


def _frame(parts):
    out = bytearray()
    for p in parts:
        h = (len(p) << 1) | 1
        out += bytes([h & 255, (h >> 8) & 255, h >> 16]) + p
    return bytes(out)


@pytest.mark.parametrize("codec", ["DEFLATE", "LZ4"])
@pytest.mark.parametrize("frames", [40, 300, 1100])
def test_every_byte_of_an_original_chunk(dev, codec, frames):
    import torch
    import paper_2307_03760_amd as codag
    rng = np.random.default_rng(frames)
    data = rng.integers(0, 256, BLOCK + max(LENGTHS), dtype=np.uint8)
    out = torch.empty(BLOCK * (frames - 2), dtype=torch.uint8, device=dev)
    out_len = torch.zeros(1, dtype=torch.int64, device=dev)
    st = torch.zeros(1, dtype=torch.int32, device=dev)
    wrong = []
    for n in LENGTHS:
        for whole in (0, 1):  # the only chunk; the last one, after a whole block
            total = whole * BLOCK + n
            want = data[:total]
            parts = [want[:BLOCK].tobytes()] * whole + [want[whole * BLOCK:].tobytes()]
            src = torch.from_numpy(np.frombuffer(_frame(parts) + b"\0" * 16, np.uint8).copy()).to(dev)[:-16]
            marked = out[:2 * BLOCK]
            marked.copy_(torch.from_numpy(~np.resize(want, 2 * BLOCK)))  # differs from the data everywhere
            codag.orc_decompress_stream(getattr(codag, codec), src, BLOCK, out, out_len, st)
            torch.cuda.synchronize()
            got = marked.cpu().numpy()
            assert int(st.item()) == 0 and int(out_len.item()) == total
            if not np.array_equal(got[:total], want):
                wrong.append((whole, n))
            assert np.array_equal(got[total:], ~np.resize(want, 2 * BLOCK)[total:])
    assert not wrong, wrong
