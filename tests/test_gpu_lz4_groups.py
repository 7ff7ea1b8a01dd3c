"""GPU parity of LZ4 launches and ORC streams with more blocks than workgroups:
every block decoded once whatever the lengths and counts, blocks set aside for
one wave (tiny, long runs, one huge field) among ordinary and damaged ones."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_parity
from test_gpu_launch_speed import _lz4_long_runs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03760_amd as codag
    codag.lib()
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def pool():
    rng = np.random.default_rng(41)
    vocab = workloads._vocab(0)
    datas = [workloads.zipf_text(int(n), rng, vocab) for n in np.exp(rng.uniform(2, 11, 40))]
    datas += [rng.bytes(int(n)) for n in np.exp(rng.uniform(1, 11, 10))] + [bytes(9), bytes(30000), b"ab" * 20000]
    out = [(workloads.lz4_block(d), len(d)) for d in datas]
    out += [_lz4_long_runs(k) for k in range(4)]
    out += [(b[:int(rng.integers(0, len(b)))], n) for b, n in out[::5]]            # cut off
    out += [(b, max(0, n - int(rng.integers(1, 9)))) for b, n in out[1:50:5]]      # too little room
    for b, n in out[2:50:4]:                                                     # damaged
        m = bytearray(b)
        m[int(rng.integers(0, len(m)))] ^= 1 << int(rng.integers(0, 8))
        out.append((bytes(m), n))
    return out


@pytest.mark.parametrize("n", [1, 200, 256, 257, 300, 511, 512, 513, 768, 1000, 1023, 1024])
def test_launches_of_every_count(dev, pool, n):
    pick = np.random.default_rng(n).integers(0, len(pool), n)
    ch = workloads._pack([oracle.LZ4] * n, [pool[k][0] for k in pick], [pool[k][1] for k in pick])
    st = assert_parity(oracle.LZ4, ch, dev, guards=n < 512)
    assert n < 200 or ((st == 0).sum() > n // 2 and (st != 0).any())


@pytest.mark.parametrize("frames", [3, 255, 300, 600, 1021])
@pytest.mark.parametrize("spare", [0, 500])
def test_streams_of_every_count(dev, frames, spare):
    """Capacities that allow more chunks than there are, too."""
    import torch
    import paper_2307_03760_amd as codag
    if frames + spare + 2 > 1024:
        pytest.skip("a wave a chunk")
    rng = np.random.default_rng(frames)
    block, vocab = 3000, workloads._vocab(0)
    kinds = [workloads.zipf_text(block, rng, vocab), rng.bytes(block), bytes(block),
             rng.bytes(1400) + workloads.zipf_text(1600, rng, vocab)]
    framed, want = bytearray(), []
    for f in range(frames):
        d = kinds[int(rng.integers(4))]
        c = workloads.lz4_block(d)
        original = len(c) >= block and f % 2 == 0
        p = d if original else c
        h = (len(p) << 1) | int(original)
        framed += bytes([h & 255, (h >> 8) & 255, h >> 16]) + p
        want.append(d)
    src = torch.from_numpy(np.frombuffer(bytes(framed) + b"\0" * 16, np.uint8).copy()).to(dev)[:-16]
    out = torch.full((block * (frames + spare),), 0xA5, dtype=torch.uint8, device=dev)
    out_len = torch.zeros(1, dtype=torch.int64, device=dev)
    st = torch.full((1,), 99, dtype=torch.int32, device=dev)
    codag.orc_decompress_stream(codag.LZ4, src, block, out, out_len, st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0 and int(out_len.item()) == block * frames
    got = out.cpu().numpy()
    assert got[:block * frames].tobytes() == b"".join(want) and (got[block * frames:] == 0xA5).all()
