"""Small launches of the streaming kernel, one workgroup per (query tile, head) or per equal piece of one
(stream_form): parts of no, one and several tiles, query tiles without queries, two query tiles of a user, tiles of
new rows in a part of their own, more pairs than CUs, and a schedule that fills a wavefront's lanes."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from helpers import draw_step_data
from test_gpu_parity import FILL, _harness, _oracle_store, check_attention
from test_gpu_stream_join import _check_all_forms

pytestmark = pytest.mark.gpu


def _step(w, data):
    step = _harness().GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    return step


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("top", [16, 31, 48, 64, 100])
@pytest.mark.parametrize("form", ["whole", "pieces", "many"])
def test_small_launches_match_oracle(form, D, top):
    """whole: 7 users x 3 heads; pieces: one of them past the whole pairs' length (95 tiles; with 100 queries two
    query tiles); many: 300 pairs where whole ones serve them (a CU takes several), else even shares."""
    long = {"whole": 700, "pieces": 3030, "many": 200}[form]
    prefix, new = [long, 5, 0, 333, 31, 64, 1], [top, 1, min(33, top), 16, 1, 0, top - 7]
    heads = 3
    if form == "many":
        prefix, new, heads = prefix * 10, new * 10, 5
    w = W.custom_workload("pieces", 60 + D + top, "bf16", 1, heads, D, 16, prefix, new, chunk_tokens=1024)
    data = draw_step_data(w)
    for check in _check_all_forms(w, _step(w, data), data):
        check()


@pytest.mark.parametrize("users,heads,long", [(64, 1, 3000), (65, 1, 3000), (1, 1, 8861), (1, 96, 2500), (1, 97, 2500)])
def test_pieces_up_to_the_lanes_and_the_pairs_of_a_schedule(users, heads, long):
    """64 users fill the lanes that hold the schedule, 65 take even shares; one pair in 31 pieces, the most there are of one; 96
    pairs and 97."""
    prefix = [long] + [int(x) for x in np.random.default_rng(7).integers(0, 90, users - 1)]
    w = W.custom_workload("lanes", 70 + users, "bf16", 1, heads, 64, 32, prefix, [3] * users, chunk_tokens=1024)
    data = draw_step_data(w)
    for check in _check_all_forms(w, _step(w, data), data):
        check()


# 95 + 89 + 82 tiles x 2 heads in pieces of 6 are 90 for up to 156 workgroups; 376 x 2 are 126 for 64
@pytest.mark.parametrize("prefix,new,whole", [([3000, 2800, 2600], [8, 20, 5], False), ([12000], [8], True)])
def test_more_pieces_than_the_stated_bounds_allow(prefix, new, whole):
    """Fewer pages stated than the users hold: their tiles make more pieces than they would, as long as there are as many
    workgroups; beyond, pairs stay whole.  A whole pair leaves nothing in the workspace but descriptors."""
    w = W.custom_workload("understated", 81, "bf16", 1, 2, 64, 16, prefix, new, chunk_tokens=1024)
    data = draw_step_data(w)
    step = _step(w, data)
    store = _oracle_store(w, data)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    step.batch.meta.total_pages = 4
    check_attention(w, step.attention(data, 0), ref)
    descriptors = 32 * 256                                          # bytes, of as many workgroups as such a launch has at most
    assert (int((step.ws != 0xA5).sum()) <= descriptors) == whole


@pytest.mark.parametrize("history", [900, 4000])                # a whole pair, and one in pieces
@pytest.mark.parametrize("D", [64, 128])
def test_a_part_with_a_far_larger_reference_and_one_with_none(D, history):
    """One key outweighs everything in the other parts, which are scaled down to nothing without overflow; the first
    48 keys weigh nothing (-inf), so that a part's first tile names no reference."""
    w = W.custom_workload("late_key", 13, "bf16", 1, 2, D, 16, [history], [40], chunk_tokens=1024)
    for late in (True, False):
        data = draw_step_data(w)
        data["q"][0] = W.f32_to_bf16_bits(np.abs(W.bf16_bits_to_f32(data["q"][0])) + 0.5)
        h = np.array(data["hist"][0][0])
        if late:
            h[0] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(h[0]) * 0.01)
            h[0, 411] = W.f32_to_bf16_bits(np.full((w.heads, w.head_dim), 60.0, np.float32))
        else:
            h[0, :48, :, 7] = W.f32_to_bf16_bits(np.full((48, w.heads), -np.inf, np.float32))
        data["hist"][0][0] = h
        step = _step(w, data)
        store = _oracle_store(w, data)
        ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
        assert np.isfinite(ref).all()
        check_attention(w, step.attention(data, 0), ref)
