"""Batched launches whose queue ends before, at and after the positions that are
dealt to the waves before they claim any: every chunk is decoded once."""
import numpy as np
import pytest

import oracle
from test_gpu_batch_rle_only import _chunks, _run, dev  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wpb,claim", [(1, 1), (2, 3), (4, 2)])
def test_queue_ends_around_the_dealt_positions(dev, wpb, claim):  # noqa: F811
    import torch
    import paper_2307_03760_amd as codag
    dealt = torch.cuda.get_device_properties(0).multi_processor_count * wpb * claim  # one workgroup a CU
    for n in (1, claim, claim + 1, dealt // wpb, dealt - 1, dealt, dealt + 1, 2 * dealt + 5):
        codecs = np.random.default_rng(n).choice([oracle.RLE_V1, oracle.RLE_V2, oracle.DEFLATE, oracle.LZ4], n)
        codecs[n // 2] = oracle.DEFLATE
        ticks = torch.zeros(n, dtype=torch.int64, device=dev)
        order = torch.from_numpy(np.random.default_rng(n + 1).permutation(n).astype(np.int32)).to(dev)
        plan = codag.Plan(order=codag.ORDER_GIVEN, waves_per_cu=wpb, waves_per_block=wpb, chunks_per_claim=claim)
        _run(plan, _chunks(codecs), dev, order=order, ticks=ticks)
        assert bool((ticks > 0).all())
