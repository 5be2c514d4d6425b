"""The fp32 attention kernel where its 16-query blocks and the 16-token sub-blocks that its eight
wavefronts take in turn begin and end, and values that a weight of zero does not cancel."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from conftest import KERNEL_PLAIN
from helpers import as_values, draw_step_data
from test_gpu_parity import FILL, _harness, _oracle_store, check_attention

pytestmark = pytest.mark.gpu

# prefix, new: one key; sub-block edges; 128-key rounds; users without tokens; blocks that start inside
# a 16-token stretch of the ragged rows; a history of many rounds
SHAPES = [([0, 15, 16, 17, 111, 127, 128, 0, 2900], [1, 1, 16, 15, 17, 1, 33, 0, 5]),
          ([0, 0, 64, 240], [0, 49, 32, 16])]


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("D,S", [(32, 16), (64, 32), (128, 64), (128, 16)])
def test_f32_matches_oracle(D, S, shape):
    G = _harness()
    w = W.custom_workload("f32_edges", 60 + D + S + shape, "f32", 1, 3, D, S, *SHAPES[shape], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    args = (store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    check_attention(w, step.attention(data, 0), oracle.attn_incremental(*args))
    inv = 1.0 / float(w.total_lens.max())
    check_attention(w, step.attention_pointwise(data, 0, inv), oracle.attn_pointwise(*args, inv))


@pytest.mark.parametrize("D,S", [(32, 16), (64, 64), (128, 32)])
def test_f32_histories_of_more_pages_than_lanes(D, S):
    """A wavefront's lanes hold the pages of its next 64 sub-blocks: histories that end around 8 x 64 of them and
    past twice as many."""
    G = _harness()
    w = W.custom_workload("f32_long", 70 + D, "f32", 1, 1, D, S, [8175, 8192, 8300, 16500], [16, 1, 20, 2], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    args = (store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    check_attention(w, step.attention(data, 0), oracle.attn_incremental(*args))


@pytest.mark.parametrize("pointwise", [False, True])
def test_f32_hidden_infinity_stays_hidden(pointwise):
    """An infinite or NaN value row of a new token reaches its own query and later ones only: the
    rows before it equal those of the step without it."""
    G = _harness()
    w = W.custom_workload("f32_inf", 5, "f32", 1, 2, 64, 16, [37], [40])
    data = draw_step_data(w)

    def outputs():
        step = G.GpuStep(w, fill_byte=FILL)
        step.unpack_histories(data, 0)
        step.append(data, 0)
        return as_values(step.attention_pointwise(data, 0, 0.01) if pointwise else step.attention(data, 0))

    plain = outputs()
    v = np.array(data["v_new"][0])
    v[21, :, 5], v[30, :, 9] = np.inf, np.nan
    data["v_new"][0] = v
    got = outputs()
    assert np.abs(got[:21] - plain[:21]).max() <= 1e-6 * np.abs(plain).max()
    assert not np.isfinite(got[21:, :, 5]).any()
    assert np.isnan(got[30:, :, 9]).all()
    keep = [d for d in range(64) if d not in (5, 9)]
    assert np.abs(got[..., keep] - plain[..., keep]).max() <= 1e-6 * np.abs(plain).max()


@pytest.mark.parametrize("D,S", [(32, 16), (64, 32), (128, 64)])
def test_f32_plain_kernel_can_be_forced(D, S, attn_tuning):
    """The plain kernel is a second implementation for this type too: it sums in another order, so
    it matches the oracle with other bits than the matrix-core kernel."""
    G = _harness()
    w = W.custom_workload("f32_plain", 80 + D, "f32", 1, 3, D, S, *SHAPES[0], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    args = (store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    inv = 1.0 / float(w.total_lens.max())
    automatic = np.array(step.attention(data, 0)), np.array(step.attention_pointwise(data, 0, inv))
    attn_tuning(kernel=KERNEL_PLAIN)
    plain = np.array(step.attention(data, 0)), np.array(step.attention_pointwise(data, 0, inv))
    for got, other, ref in zip(plain, automatic, (oracle.attn_incremental(*args), oracle.attn_pointwise(*args, inv))):
        check_attention(w, got, ref)
        assert (got != other).any()


# users of a few keys, by the hundred: lengths of one page and of two, one with more new tokens; and as many that are too long
MANY = {"short": ([0, 3, 6, 1, 9, 0, 4], [1, 1, 2, 1, 1, 2, 1], True), "too_long": ([90, 70, 110], [1, 2, 1], False)}


@pytest.mark.parametrize("name", list(MANY))
@pytest.mark.parametrize("D,S", [(32, 16), (64, 64), (128, 16)])
def test_f32_many_short_users_take_the_plain_kernel(D, S, name, attn_tuning):
    """A workgroup of the matrix-core kernel costs the same for 8 keys as for 128 (f32_takes_plain): calls of many
    short users are the plain kernel's, with its bits, and match the oracle."""
    G = _harness()
    prefix, new, plain_taken = MANY[name]
    w = W.custom_workload("f32_many", 90 + D, "f32", 1, 8, D, S, prefix * 60, new * 60, chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    args = (store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    inv = 1.0 / float(w.total_lens.max())
    automatic = np.array(step.attention(data, 0)), np.array(step.attention_pointwise(data, 0, inv))
    attn_tuning(kernel=KERNEL_PLAIN)
    plain = np.array(step.attention(data, 0)), np.array(step.attention_pointwise(data, 0, inv))
    for got, other, ref in zip(automatic, plain, (oracle.attn_incremental(*args), oracle.attn_pointwise(*args, inv))):
        check_attention(w, got, ref)
        assert (got == other).all() == plain_taken


@pytest.mark.parametrize("scale", [1e10, 1e30])
@pytest.mark.parametrize("D,S", [(32, 16), (64, 64), (128, 32)])
def test_f32_logits_beyond_the_exponents_whole_numbers(D, S, scale):
    """Logits whose unit in the last place is many times the exponential's range: a row is its largest key's value, from
    one wavefront's keys and from several's."""
    G = _harness()
    w = W.custom_workload("f32_large", 95 + D, "f32", 1, 3, D, S, *SHAPES[0], chunk_tokens=1024)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr, sm_scale=scale)
    got = step.attention(data, 0, sm_scale=scale)
    assert np.isfinite(got).all()
    check_attention(w, got, ref)
