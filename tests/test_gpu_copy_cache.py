"""A scatter of more than the last-level cache moves its rows past it; each of its layers alone, and two of them, less so."""
import numpy as np
import pytest

import paper_2604_22881_amd as mts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,heads,head_dim", [("bf16", 8, 64), ("bf16", 16, 32), ("f32", 2, 128)])
def test_layers_in_one_launch_and_one_by_one_agree(dtype, heads, head_dim):
    import torch
    from paper_2604_22881_amd.runtime import DeviceBatch, PagedKVCache, SegmentList
    layers, page, dev = 4, 16, "cuda:0"
    es = 4 if dtype == "f32" else 2
    row = 2 * heads * head_dim * es
    prefix = np.array([30011, 14003, 150, 5], np.int32) * (2048 // row)
    need = -(-(prefix.astype(np.int64) + 1) // page)
    indptr = np.concatenate([[0], np.cumsum(need)]).astype(np.int32)
    indices = np.random.default_rng(3).permutation(indptr[-1]).astype(np.int32)
    batch = DeviceBatch(indptr, indices, prefix, np.arange(5), dev)
    segs = SegmentList.for_histories(np.arange(4), prefix, 1024, dev)
    assert segs.total_tokens * row * layers >= 336 << 20 > segs.total_tokens * row
    staging = torch.randint(-2 ** 31, 2 ** 31 - 1, (layers, segs.total_tokens * row // 4), dtype=torch.int32, device=dev)
    pools = []
    for at_once in (4, 2, 1):
        cache = PagedKVCache(layers, int(indptr[-1]), page, heads, head_dim, dtype, dev)
        cache.pool.zero_()
        for l in range(0, layers, at_once):
            mts.mts_kv_unpack_layers(cache.desc, l, at_once, staging[l], segs.total_tokens * row, *segs.args(), batch.meta)
        pools.append(cache.pool)
    assert bool((pools[0] != 0).any()) and torch.equal(pools[0], pools[1]) and torch.equal(pools[0], pools[2])
