"""The dense-prefill kernel where its pieces begin and end: blocks of one to a few tiles (fewer than
the stages in flight), users that end inside a wavefront, a tile and a block, prefixes around them,
every page size, and more (user, head) pairs than one group of an XCD holds."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from conftest import KERNEL_PREFILL
from helpers import as_values, draw_step_data
from test_gpu_parity import FILL, _harness, _oracle_store, check_attention

pytestmark = pytest.mark.gpu

SHAPES = {
    # name: (heads, prefix, new)
    "few_tiles": (3, [0, 0, 0, 0, 0, 31, 64, 95], [1, 32, 33, 65, 97, 1, 32, 33]),
    "block_ends": (2, [0, 0, 0, 17, 160], [127, 129, 257, 255, 300]),
    "many_pairs": (5, [0, 9, 0, 40, 0, 0, 3, 0, 70, 0, 0, 0, 5], [140, 30, 1, 60, 33, 270, 8, 0, 64, 90, 16, 128, 200]),
}


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("D,S", [(64, 16), (64, 64), (128, 16), (128, 32)])
@pytest.mark.parametrize("name", list(SHAPES))
def test_prefill_blocks_match_oracle(name, D, S, split, attn_tuning):
    attn_tuning(kernel=KERNEL_PREFILL, **(dict(min_tiles=1, max_waves=64, pair_cost=1) if split else {}))
    G = _harness()
    heads, prefix, new = SHAPES[name]
    w = W.custom_workload(name, 500 + D + S, "bf16", 1, heads, D, S, prefix, new, chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    args = (store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    check_attention(w, step.attention(data, 0), oracle.attn_incremental(*args))
    inv = 1.0 / float(w.total_lens.max())
    check_attention(w, step.attention_pointwise(data, 0, inv), oracle.attn_pointwise(*args, inv))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name,heads,new", [("equal", 5, [140] * 13), ("unequal", 5, [300] + [70] * 12), ("one_pair", 1, [150, 20]),
                                            ("long", 9, [1100, 3, 3])])
def test_order_of_the_blocks_does_not_matter(name, heads, new, D, attn_tuning):
    """How many (user, head) pairs an XCD takes at a time depends on how much K/V the call states and on
    how unequal its segments are: every block is worked on once whatever the order, with the same bits."""
    attn_tuning(kernel=KERNEL_PREFILL)
    G = _harness()
    w = W.custom_workload(name, 600 + D + heads, "bf16", 1, heads, D, 16, [40] * len(new), new, chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.ws_bytes = 0                                              # one workgroup per block
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    few = np.array(step.attention(data, 0))                        # all of an XCD's pairs at a time
    check_attention(w, few, oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens,
                                                    w.new_indptr))
    step.batch.meta.total_pages = 1 << 20                          # groups of pairs
    assert np.array_equal(few, np.array(step.attention(data, 0)))


@pytest.mark.parametrize("D", [64, 128])
def test_prefill_redoes_a_block_whose_reference_overflows(D, attn_tuning):
    """A far larger key behind the first tile: the block goes round again with the exact max, all its
    stages fetched anew."""
    attn_tuning(kernel=KERNEL_PREFILL)
    G = _harness()
    w = W.custom_workload("late_key", 13, "bf16", 1, 2, D, 16, [300, 0], [40, 260])
    data = draw_step_data(w)
    h = np.array(data["hist"][0][0])
    h[0] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(h[0]) * 0.01)
    h[0, 211] = W.f32_to_bf16_bits(np.full((w.heads, w.head_dim), 60.0, np.float32))
    data["hist"][0][0] = h
    data["q"][0] = W.f32_to_bf16_bits(np.abs(W.bf16_bits_to_f32(data["q"][0])) + 0.5)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    got = step.attention(data, 0)
    assert np.isfinite(as_values(got)).all()
    check_attention(w, got, ref)
