"""Share boundaries that the streaming kernel closes inside a workgroup, where the launch is large enough or
its pairs have many pieces (joins_pieces): pairs that end in the next wavefront's share, span several
wavefronts, whole workgroups or several of them, pairs cut inside their schedule allowance; and the
per-wavefront partials of the other launches and of schedules of very many users."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from conftest import KERNEL_PREFILL, KERNEL_STREAMING
from helpers import as_values, draw_step_data
from test_gpu_parity import FILL, _harness, _oracle_store, check_attention

pytestmark = pytest.mark.gpu

# shares of one to a few tiles over 95-tile, 22-tile and single-tile pairs; launches of one workgroup,
# of few, and of as many as the shares fill; allowances that shares begin and end in
PLANS = [dict(min_tiles=1, pair_cost=1), dict(min_tiles=2, pair_cost=3), dict(min_tiles=5, pair_cost=9),
         dict(max_waves=4, pair_cost=1), dict(max_waves=28, pair_cost=4), dict(min_tiles=2 ** 31 - 1), {}]


def _check_all_forms(w, step, data):
    store = _oracle_store(w, data)
    args = (store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    ref = oracle.attn_incremental(*args)
    inv = 1.0 / float(w.total_lens.max())
    pw = oracle.attn_pointwise(*args, inv)
    yield lambda: check_attention(w, step.attention_unappended(data, 0), ref)
    yield lambda: check_attention(w, step.attention(data, 0), ref)
    yield lambda: check_attention(w, step.attention_pointwise(data, 0, inv), pw)
    yield lambda: check_attention(w, step.attention_unappended(data, 0, inv_norm=inv), pw)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("top", [16, 40, 64])
def test_joined_pieces_match_oracle(D, top, attn_tuning):
    import torch
    import paper_2604_22881_amd as mts
    G = _harness()
    w = W.custom_workload("join", 40 + D + top, "bf16", 1, 3, D, 16, [3030, 5, 0, 700, 31, 64, 1],
                          [top, 1, min(33, top), 16, 1, 0, top - 7], chunk_tokens=1024)
    data = draw_step_data(w)
    attn_tuning(kernel=KERNEL_STREAMING)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    for check in _check_all_forms(w, step, data):
        for plan in PLANS:
            attn_tuning(kernel=KERNEL_STREAMING, **plan)
            need = mts.mts_attn_workspace_bytes(step.cache.desc, step.batch.meta)
            if need > step.ws_bytes:
                step.ws, step.ws_bytes = torch.full((need,), 0xA5, dtype=torch.uint8, device=G.DEV), need
            check()


@pytest.mark.parametrize("users,top", [(64, 3), (65, 3), (32, 90), (33, 90), (1, 1)])
@pytest.mark.parametrize("plan", [PLANS[0], PLANS[3], PLANS[4]])
def test_schedule_up_to_the_lanes_of_a_wavefront(plan, users, top, attn_tuning):
    """64 (user, query tile)s are scheduled in the lanes, more through LDS; users without new tokens and query tiles
    without queries among them, in the first and the last lanes too."""
    rng = np.random.default_rng(users + top)
    prefix = [int(x) for x in rng.integers(0, 200, users)]
    new = [int(x) for x in rng.integers(0, 4, users)]
    new[0], new[-1] = 0, 0
    new[users // 2] = top
    attn_tuning(kernel=KERNEL_STREAMING, **plan)
    w = W.custom_workload("lanes", 90 + users, "bf16", 1, 2, 64, 16, prefix, new, chunk_tokens=1024)
    data = draw_step_data(w)
    step = _harness().GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    for check in _check_all_forms(w, step, data):
        check()


@pytest.mark.parametrize("heads", [2, 32])              # 32: enough wavefronts to fold inside workgroups
def test_joined_piece_with_a_far_larger_reference(heads, attn_tuning):
    """One piece of a cut pair holds a key that outweighs everything in the others: the fold scales
    them down to nothing without overflow."""
    attn_tuning(kernel=KERNEL_STREAMING, min_tiles=2, pair_cost=1)
    G = _harness()
    w = W.custom_workload("late_key", 13, "bf16", 1, heads, 64, 16, [900], [40])
    data = draw_step_data(w)
    h = np.array(data["hist"][0][0])
    h[0] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(h[0]) * 0.01)
    h[0, 411] = W.f32_to_bf16_bits(np.full((w.heads, w.head_dim), 60.0, np.float32))
    data["hist"][0][0] = h
    data["q"][0] = W.f32_to_bf16_bits(np.abs(W.bf16_bits_to_f32(data["q"][0])) + 0.5)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    store = _oracle_store(w, data)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    got = step.attention(data, 0)
    assert np.isfinite(as_values(got)).all()
    check_attention(w, got, ref)


@pytest.mark.parametrize("min_tiles", [3, 5, 8])
@pytest.mark.parametrize("heads", [2, 128])             # 128: enough wavefronts to fold inside workgroups
@pytest.mark.parametrize("D", [64, 128])
def test_pieces_after_a_first_tile_that_weighs_nothing(D, heads, min_tiles, attn_tuning):
    """The first 48 tokens have logit -inf for every query (infinite keys): a piece whose first tile names
    no reference still counts when the pieces are joined or merged."""
    attn_tuning(kernel=KERNEL_STREAMING, min_tiles=min_tiles, pair_cost=1)
    G = _harness()
    w = W.custom_workload("silent_start", 15, "bf16", 1, heads, D, 16, [900], [40])
    data = draw_step_data(w)
    data["q"][0] = W.f32_to_bf16_bits(np.abs(W.bf16_bits_to_f32(data["q"][0])) + 0.5)
    h = np.array(data["hist"][0][0])
    h[0, :48, :, 7] = W.f32_to_bf16_bits(np.full((48, w.heads), -np.inf, np.float32))
    data["hist"][0][0] = h
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    store = _oracle_store(w, data)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    assert np.isfinite(ref).all()
    check_attention(w, step.attention(data, 0), ref)


@pytest.mark.parametrize("users", [1300, 4090])
def test_schedule_of_many_users_leaves_no_room_to_join(users, attn_tuning):
    """head_dim 128, 64-query tiles: the schedule (4 words a user) and the handed-over pieces (108 KB, 96
    pointwise) do not fit the LDS together beyond about 1100 users unappended, 3320 from the pool and 4087
    pointwise from the pool."""
    attn_tuning(kernel=KERNEL_STREAMING)
    G = _harness()
    rng = np.random.default_rng(3)
    prefix, new = rng.integers(0, 12, users), np.ones(users, np.int64)
    prefix[[3, 700]], new[[3, 5, 700]] = (1500, 400), (64, 50, 33)
    w = W.custom_workload("many", 9, "bf16", 1, 1, 128, 16, list(prefix), list(new), chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    for check in _check_all_forms(w, step, data):
        check()


@pytest.mark.parametrize("D,new", [(32, 20), (64, 32), (128, 1), (128, 32), (128, 50)])
def test_automatic_shares_are_cut_at_four_tiles(D, new, attn_tuning):
    """Where a call is cut decides how its weights round: the automatic cut is the same for every head
    and query size, so that results do not change from one release to the next."""
    G = _harness()
    w = W.custom_workload("cuts", 21 + D + new, "bf16", 1, 2, D, 32, [2000], [new], chunk_tokens=1024)
    data = draw_step_data(w)

    def attention(**plan):
        attn_tuning(kernel=KERNEL_STREAMING, **plan)
        step = G.GpuStep(w, fill_byte=FILL)
        step.unpack_histories(data, 0)
        step.append(data, 0)
        return np.array(step.attention(data, 0))

    assert (attention() == attention(min_tiles=4)).all()
    assert (attention() != attention(min_tiles=3)).any()


@pytest.mark.parametrize("kernel,D,max_waves,heads", [(KERNEL_STREAMING, 64, 4, 1), (KERNEL_STREAMING, 128, 4, 1),
                                                      (KERNEL_STREAMING, 32, 32, 1), (KERNEL_PREFILL, 64, 16, 1),
                                                      (KERNEL_PREFILL, 128, 16, 1)])
def test_sum_of_pieces_overflows_though_none_of_them_does(kernel, D, max_waves, heads, attn_tuning):
    """Every piece of a cut pair holds one key of weight 2^120.7 to 2^121.7 against its reference, and values of
    64 in one dim: 1.7e38 to 2.8e38 in a piece, beyond the fp32 range (3.4e38) in two.  32 wavefronts at
    head_dim 32 fold inside workgroups (joins_pieces), the others leave their pieces to the merge."""
    tiles, cost = 248, 8
    attn_tuning(kernel=kernel, max_waves=max_waves, pair_cost=cost, min_tiles=4)
    shares = max_waves // 4 if kernel == KERNEL_PREFILL else max_waves
    G = _harness()
    w = W.custom_workload("far_keys", 17, "bf16", 1, heads, D, 16, [tiles * 32 - 8], [8], chunk_tokens=1024)
    data = draw_step_data(w)
    k, v = np.zeros_like(W.bf16_bits_to_f32(np.array(data["hist"][0][0])))
    x = np.float32(121.2 / (np.log2(np.e) * 16 / np.sqrt(D)))       # times a query of 16 / sqrt(D): 121.2 in base 2
    far = [s * (tiles + cost) // shares - cost + (tiles + cost) // shares // 2 for s in range(shares)]
    far = [t for t in far if t > 0]                                 # the allowance comes before the first tile
    for t in far:
        k[t * 32 + 5, :, 3] = x
    v[:, :, 7] = 64.0
    data["hist"][0][0] = W.f32_to_bf16_bits(np.stack([k, v]))
    data["k_new"][0] = W.f32_to_bf16_bits(np.zeros_like(W.bf16_bits_to_f32(data["k_new"][0])))
    data["v_new"][0] = data["k_new"][0].copy()
    q = np.zeros_like(W.bf16_bits_to_f32(data["q"][0]))
    q[..., 3] = 16.0
    data["q"][0] = W.f32_to_bf16_bits(q)
    log2_weight = float(W.bf16_bits_to_f32(W.f32_to_bf16_bits(np.array([x]))).item()) * 16 / np.sqrt(D) * np.log2(np.e)
    assert 120.7 < log2_weight < 121.7 and 64 * 2 ** log2_weight < 3.0e38
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    store = _oracle_store(w, data)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    assert np.allclose(ref[:, 0, 7], 64.0)
    check_attention(w, step.attention(data, 0), ref)
