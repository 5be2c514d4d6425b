"""The split launch of the dense-prefill kernel (long new segments, work cut evenly over a persistent
launch): shares that cut blocks once, many times and not at all, shares that walk through several
blocks, heads and users, users without new tokens, pieces without a visible key, every workspace size."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from conftest import KERNEL_PREFILL
from helpers import as_values, draw_step_data
from test_gpu_parity import FILL, _harness, _oracle_store, check_attention

pytestmark = pytest.mark.gpu

CASES = {
    # name: (D, S, prefix, new)
    "one_user": (128, 16, [0], [389]),                            # 128-query blocks, a ragged last one
    "one_user_d64": (64, 32, [31], [513]),                        # 256-query blocks
    "mixed": (128, 32, [1500, 0, 700, 33, 0], [8, 300, 0, 1, 127]),
    "mixed_d64": (64, 64, [0, 1291, 5, 640], [600, 17, 0, 64]),
}
SPLITS = {
    "one_step_shares": dict(min_tiles=1, max_waves=1024, pair_cost=1),
    "one_workgroup": dict(max_waves=4),
    "odd_shares": dict(min_tiles=3, max_waves=28, pair_cost=7),
    "xcd_shares": dict(min_tiles=2, max_waves=32),
    "least_share_past_every_step": dict(min_tiles=1 << 30, max_waves=64),
}


def _workload(name):
    D, S, prefix, new = CASES[name]
    return W.custom_workload(name, 300 + len(name), "bf16", 1, 2, D, S, prefix, new, chunk_tokens=1024)


@pytest.mark.parametrize("split", list(SPLITS))
@pytest.mark.parametrize("name", list(CASES))
def test_split_prefill_matches_oracle(name, split, attn_tuning):
    attn_tuning(kernel=KERNEL_PREFILL, **SPLITS[split])
    G, w = _harness(), _workload(name)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    assert step.ws_bytes > 0
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    check_attention(w, step.attention(data, 0), ref)
    inv = 1.0 / float(w.total_lens.max())
    ref = oracle.attn_pointwise(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr, inv)
    check_attention(w, step.attention_pointwise(data, 0, inv), ref)


# A cut block weighs its keys against the reference of the uncut one, so that split and unsplit results
# differ by the order of fp32 sums alone: the sum of a row's w * v (a few hundred to a few thousand terms) moves by
# about 1e-6 of sum |w * v|, which is at most 60 times the row's root mean square here, and a bf16 output is
# rounded the other way only within that distance of a tie: about 1e-6 * 60 / 2^-8 = 1.5 % of the values
# if every sum moved that far, by one unit in the last place (2^-7 of the value).  References of the pieces' own
# round all weights anew: 4 to 45 % of the values differ.
def _same_but_for_fp32_order(a, b):
    rms = np.sqrt((b * b).mean())
    assert (a != b).mean() <= 0.015
    assert (np.abs(a - b) <= 2.0 ** -7 * np.maximum(np.abs(a), np.abs(b)) + 6e-5 * rms).all()


@pytest.mark.parametrize("split", list(SPLITS))
@pytest.mark.parametrize("name", list(CASES))
def test_split_prefill_equals_unsplit(name, split, attn_tuning):
    import torch
    import paper_2604_22881_amd as mts
    attn_tuning(kernel=KERNEL_PREFILL, **SPLITS[split])
    G, w = _harness(), _workload(name)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    got = as_values(step.attention(data, 0))
    q = G.to_dev(data["q"][0])
    out = torch.full((w.total_new, w.heads, w.head_dim), -1, dtype=q.dtype, device=G.DEV)
    mts.mts_attn_incremental(step.cache.desc, 0, q, out, step.batch.meta, 0.0, None, 0)     # no room to split
    torch.cuda.synchronize()
    _same_but_for_fp32_order(got, as_values(G.to_host(out, w.np_dtype)))


@pytest.mark.parametrize("heads", [5, 8, 30])                   # shares of 2 and 1 steps, of 3 and 1 or 4 and 2, of 10 to 13 and 5 to 7
@pytest.mark.parametrize("D", [64, 128])
def test_unequal_shares_of_a_full_launch(D, heads, attn_tuning):
    """A launch that fills the chip gives a CU two neighbouring shares, the first of them larger."""
    attn_tuning(kernel=KERNEL_PREFILL, min_tiles=1, max_waves=2048, pair_cost=1)
    w = W.custom_workload("unequal", 310 + D + heads, "bf16", 1, heads, D, 16, [1500, 0, 700, 0], [8, 600, 200, 0], chunk_tokens=1024)
    data = draw_step_data(w)
    step = _harness().GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    check_attention(w, step.attention(data, 0), ref)


@pytest.mark.parametrize("heads", [5, 8, 30])
@pytest.mark.parametrize("D", [64, 128])
def test_unequal_shares_equal_unsplit(D, heads, attn_tuning):
    """... whose results, softmax and pointwise, are those of uncut blocks but for the order of sums."""
    import torch
    import paper_2604_22881_amd as mts
    attn_tuning(kernel=KERNEL_PREFILL, min_tiles=1, max_waves=2048, pair_cost=1)
    G = _harness()
    w = W.custom_workload("unequal", 310 + D + heads, "bf16", 1, heads, D, 16, [1500, 0, 700, 0], [8, 600, 200, 0], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    q = G.to_dev(data["q"][0])
    inv = 1.0 / float(w.total_lens.max())
    ref = oracle.attn_pointwise(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr, inv)
    softmax, pointwise = step.attention(data, 0), step.attention_pointwise(data, 0, inv)
    check_attention(w, pointwise, ref)
    whole = [torch.full((w.total_new, w.heads, w.head_dim), -1, dtype=q.dtype, device=G.DEV) for _ in range(2)]
    mts.mts_attn_incremental(step.cache.desc, 0, q, whole[0], step.batch.meta, 0.0, None, 0)
    mts.mts_attn_pointwise(step.cache.desc, 0, q, whole[1], step.batch.meta, inv, 0.0, None, 0)
    torch.cuda.synchronize()
    for got, want in zip((softmax, pointwise), whole):
        _same_but_for_fp32_order(as_values(got), as_values(G.to_host(want, w.np_dtype)))


@pytest.mark.parametrize("users,heads,long", [(64, 1, 300), (65, 1, 300), (200, 2, 300), (1024, 1, 300), (2, 70, 260), (1, 1, 8400)])
def test_schedule_in_the_lanes_of_a_wavefront(users, heads, long, attn_tuning):
    """One user a lane, groups of users behind a lane (2, 4 and 16 of them), more heads and more query blocks than lanes."""
    attn_tuning(kernel=KERNEL_PREFILL, min_tiles=2, max_waves=512)
    G = _harness()
    rng = np.random.default_rng(users)
    prefix, new = [int(x) for x in rng.integers(0, 70, users)], [int(x) for x in rng.integers(0, 4, users)]
    new[users * 2 // 3] = long
    w = W.custom_workload("lanes", 90 + users, "bf16", 1, heads, 128, 64, prefix, new, chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    check_attention(w, step.attention(data, 0), ref)


def test_split_prefill_block_whose_first_keys_weigh_nothing(attn_tuning):
    """Infinite keys: the first 48 tokens have logit -inf for every query, so the first tile names no
    reference; the pieces of the later tiles still count."""
    attn_tuning(kernel=KERNEL_PREFILL, min_tiles=2, max_waves=64, pair_cost=1)
    G = _harness()
    w = W.custom_workload("silent_start", 14, "bf16", 1, 2, 64, 16, [300, 0], [40, 270])
    data = draw_step_data(w)
    data["q"][0] = W.f32_to_bf16_bits(np.abs(W.bf16_bits_to_f32(data["q"][0])) + 0.5)
    h = np.array(data["hist"][0][0])
    h[0, :48, :, 7] = W.f32_to_bf16_bits(np.full((48, w.heads), -np.inf, np.float32))
    data["hist"][0][0] = h
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    assert np.isfinite(ref).all()
    check_attention(w, step.attention(data, 0), ref)


def test_split_prefill_with_less_or_no_workspace():
    """A call that would split runs with any workspace: fewer shares, then none, the same result."""
    import torch
    import paper_2604_22881_amd as mts
    G = _harness()
    w = W.custom_workload("little_room", 11, "bf16", 1, 2, 64, 16, [0, 2200], [1300, 40], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    store = _oracle_store(w, data)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    assert step.ws_bytes > 0
    full, q = step.ws_bytes, G.to_dev(data["q"][0])
    for ws, nbytes in ((step.ws, full), (step.ws, full // 3), (step.ws, 1000), (step.ws[16:], full - 16), (None, 0)):
        out = torch.full((w.total_new, w.heads, w.head_dim), -1, dtype=q.dtype, device=G.DEV)
        mts.mts_attn_incremental(step.cache.desc, 0, q, out, step.batch.meta, 0.0, ws, nbytes)
        torch.cuda.synchronize()
        check_attention(w, G.to_host(out, w.np_dtype), ref)


def test_split_prefill_redoes_a_piece_whose_reference_overflows(attn_tuning):
    """The reference max of a block comes from its first tile; a far larger key in a later
    piece overflows the weights and the piece is redone with the exact max before the merge."""
    attn_tuning(kernel=KERNEL_PREFILL, min_tiles=8, max_waves=64)
    G = _harness()
    w = W.custom_workload("late_key", 13, "bf16", 1, 2, 128, 16, [900, 0], [40, 260])
    data = draw_step_data(w)
    h = np.array(data["hist"][0][0])
    h[0] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(h[0]) * 0.01)
    h[0, 411] = W.f32_to_bf16_bits(np.full((w.heads, w.head_dim), 60.0, np.float32))
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


# The queries' rooms lie behind the page table, or inside its end where two workgroups fit a CU only so: the last length in front
# of that range, its first, one within, its last, the first past it (head_dim 64: its first).
@pytest.mark.parametrize("D,tokens", [(128, 97984), (128, 97985), (128, 114000), (128, 130752), (128, 130753), (64, 147137)])
def test_split_prefill_of_a_page_table_around_the_queries_rooms(D, tokens, attn_tuning):
    import torch
    import paper_2604_22881_amd as mts
    attn_tuning(kernel=KERNEL_PREFILL, max_waves=12)
    G = _harness()
    w = W.custom_workload("long_table", 17, "bf16", 1, 1, D, 16, [tokens - 300], [300], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    assert step.ws_bytes > 0
    step.unpack_histories(data, 0)
    step.append(data, 0)
    got = as_values(step.attention(data, 0))
    q = G.to_dev(data["q"][0])
    out = torch.full((w.total_new, w.heads, w.head_dim), -1, dtype=q.dtype, device=G.DEV)
    mts.mts_attn_incremental(step.cache.desc, 0, q, out, step.batch.meta, 0.0, None, 0)     # no overlap at these lengths
    torch.cuda.synchronize()
    want = as_values(G.to_host(out, w.np_dtype))
    # Sums of 1e5 terms in fp32 move by up to sqrt(1e5) 2^-24 = 2e-5 of sum |w v|, which is sqrt(1e5) 0.8 = 250 times an
    # average of independent values: 5e-3 of the result's root mean square, and a unit of bf16.  Ids of other pages in a
    # wavefront's room (512 of up to 8176) would change the average by sqrt(2 / 16) = 0.35 of it.
    rms = np.sqrt((want * want).mean())
    assert (np.abs(got - want) <= 2.0 ** -7 * np.maximum(np.abs(got), np.abs(want)) + 5e-3 * rms).all()


# Blocks whose own ids reach into the queries' rooms, one workgroup taking them whole: the last id in the room of each
# wavefront, of 512 words from id 6128 on at head_dim 128 (the split softmax form's alone), of 1280 from 9200 (split softmax) and of 1024
# from 10224 (pointwise and unsplit) at 64, up to the last table that overlaps.
@pytest.mark.parametrize("D,ids", [(64, 10300), (64, 11300), (64, 12300), (64, 14316), (128, 6300), (128, 6800), (128, 7400), (128, 8172)])
def test_page_ids_in_every_wavefronts_room(D, ids, attn_tuning):
    """The same keys in pages of 64 tokens, whose table is a quarter as long and lies beside the rooms: the same bits."""
    import torch
    import paper_2604_22881_amd as mts
    attn_tuning(kernel=KERNEL_PREFILL, max_waves=4)
    G = _harness()
    outs, data = [], None
    for S in (16, 64):
        w = W.custom_workload("long_table", 19, "bf16", 1, 1, D, S, [16 * ids - 305], [300], chunk_tokens=1 << 20)
        data = draw_step_data(w) if data is None else data
        step = G.GpuStep(w, fill_byte=FILL)
        assert step.ws_bytes > 0
        step.unpack_histories(data, 0)
        step.append(data, 0)
        q, got = G.to_dev(data["q"][0]), []
        for pointwise in (False, True):
            for ws, nbytes in ((step.ws, step.ws_bytes), (None, 0)):                        # split, unsplit
                out = torch.full((w.total_new, w.heads, w.head_dim), -1, dtype=q.dtype, device=G.DEV)
                if pointwise:
                    mts.mts_attn_pointwise(step.cache.desc, 0, q, out, step.batch.meta, 1.0 / 300, 0.0, ws, nbytes)
                else:
                    mts.mts_attn_incremental(step.cache.desc, 0, q, out, step.batch.meta, 0.0, ws, nbytes)
                torch.cuda.synchronize()
                got.append(G.to_host(out, w.np_dtype))
        outs.append(got)
    for form, a, b in zip(("split", "unsplit", "pointwise split", "pointwise unsplit"), *outs):
        assert np.isfinite(as_values(b)).all() and np.array_equal(a, b), form
