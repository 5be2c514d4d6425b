"""The data-movement kernel where its pieces begin and end: short and long appends (128 new tokens of
one user switch the launch) that start and end at every kind of place inside a 16-token sub-block,
head counts that do not divide a workgroup's four units, and pages that the pool does not have."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from helpers import draw_step_data
from test_gpu_parity import FILL, _harness, _oracle_store

pytestmark = pytest.mark.gpu

NEW = {"short": [1, 16, 15, 17, 33, 0, 127, 2], "long": [1, 16, 128, 131, 33, 0, 300, 2]}
PREFIX = [0, 16, 1, 15, 31, 7, 5, 30]


@pytest.mark.parametrize("new", list(NEW))
@pytest.mark.parametrize("dtype,H,D,S", [("bf16", 1, 128, 16), ("bf16", 5, 64, 32), ("bf16", 7, 32, 64),
                                         ("f32", 3, 128, 16), ("f32", 6, 32, 32)])
def test_append_at_sub_block_edges(dtype, H, D, S, new):
    G = _harness()
    w = W.custom_workload("edges", 900 + H + D, dtype, 1, H, D, S, PREFIX, NEW[new], chunk_tokens=13)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    store = _oracle_store(w, data)
    assert np.array_equal(step.pool_image(0), G.expected_pool_image(w, store, 0, FILL))
    users = [u for u in range(w.batch) if w.total_lens[u]]
    pos = [u % 3 if w.total_lens[u] > 3 else 0 for u in users]
    cnt = [int(w.total_lens[u]) - p for u, p in zip(users, pos)]
    for u, p, n, g in zip(users, pos, cnt, step.pack(0, users, pos, cnt)):
        assert g.tobytes() == oracle.pack(store, 0, w.user_pages(u), p, n).tobytes(), f"user {u}"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_every_range_inside_a_sub_block_is_stored(dtype, D):
    """A partly covered sub-block's values go in the widest aligned pieces: every first and last token, in a
    launch whose K and V wavefronts are apart if the rows are wide enough."""
    G = _harness()
    ranges = [(lo, hi) for lo in range(16) for hi in range(lo + 1, 17)]
    w = W.custom_workload("ranges", 77 + D, dtype, 1, 3, D, 16, [lo for lo, _ in ranges], [hi - lo for lo, hi in ranges], chunk_tokens=16)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    assert np.array_equal(step.pool_image(0), G.expected_pool_image(w, _oracle_store(w, data), 0, FILL))


@pytest.mark.parametrize("users", [3, 64, 65, 300])
@pytest.mark.parametrize("dtype,H,D", [("bf16", 3, 128), ("f32", 5, 32)])
def test_append_of_one_long_user_among_short_ones(users, dtype, H, D):
    """Workgroups numbered through the users' rows: users without rows, with rows that end inside and at
    sub-blocks, one long one in the middle, more of them than lanes, and as many as two rounds of lanes."""
    G = _harness()
    rng = np.random.default_rng(users)
    new = [int(x) for x in rng.integers(0, 40, users)]
    new[users // 2] = 12000 if users < 64 else 2500
    prefix = [int(x) for x in rng.integers(0, 40, users)]
    w = W.custom_workload("flat", 79 + users, dtype, 1, H, D, 16, prefix, new, chunk_tokens=64)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    assert np.array_equal(step.pool_image(0), G.expected_pool_image(w, _oracle_store(w, data), 0, FILL))


def test_more_heads_than_a_multiplication_divides_by():
    G = _harness()
    w = W.custom_workload("heads", 78, "bf16", 1, 24000, 32, 16, [3], [2], chunk_tokens=16)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    assert np.array_equal(step.pool_image(0), G.expected_pool_image(w, _oracle_store(w, data), 0, FILL))


@pytest.mark.parametrize("new", [40, 200])
@pytest.mark.parametrize("page", [-1, 1 << 20])
def test_rows_of_a_page_outside_the_pool_go_nowhere(page, new):
    """The kernel checks every page id: rows for one that the pool does not have are dropped, all
    others are stored."""
    import torch
    G = _harness()
    w = W.custom_workload("bad_page", 31, "bf16", 1, 2, 64, 16, [5, 9], [new, new], chunk_tokens=64)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.append(data, 0)
    want = step.pool_image(0).reshape(w.num_pages, -1).copy()
    lost = int(w.page_indices[1])                             # user 0's second page
    want[lost] = FILL
    again = G.GpuStep(w, fill_byte=FILL)
    again.batch.page_indices[1] = page
    torch.cuda.synchronize()
    again.append(data, 0)
    assert np.array_equal(again.pool_image(0).reshape(w.num_pages, -1), want)


@pytest.mark.parametrize("dtype,H,D", [("bf16", 3, 64), ("f32", 5, 32)])
def test_append_of_one_long_user_over_several_layers(dtype, H, D):
    """Workgroups numbered through the users' rows, over layers of a larger cache whose row buffers lie a padded stride
    apart: those layers hold the oracle's rows, the others are untouched."""
    import torch
    import paper_2604_22881_amd as mts
    G = _harness()
    L, lo, count = 5, 1, 3
    rng = np.random.default_rng(81)
    new = [int(x) for x in rng.integers(0, 40, 70)]
    new[33] = 700
    prefix = [int(x) for x in rng.integers(0, 40, 70)]
    w = W.custom_workload("flat_layers", 81, dtype, L, H, D, 32, prefix, new, chunk_tokens=64)
    data = draw_step_data(w, layers=range(lo, lo + count))
    step = G.GpuStep(w, fill_byte=FILL)
    for l in range(lo, lo + count):
        step.unpack_histories(data, l)
    n = w.total_new * H * D
    stride = n + 40                                           # elements; 80 or 160 bytes of padding
    rows = {kv: np.zeros(count * stride, dtype=w.np_dtype) for kv in ("k_new", "v_new")}
    for kv, to in rows.items():
        for i in range(count):
            to[i * stride:i * stride + n] = np.ascontiguousarray(data[kv][lo + i]).reshape(-1)
    mts.mts_kv_append_layers(step.cache.desc, lo, count, G.to_dev(rows["k_new"]), G.to_dev(rows["v_new"]),
                             stride * w.elem_bytes, step.batch.meta)
    torch.cuda.synchronize()
    store = _oracle_store(w, data, do_append=True)
    for l in range(L):
        assert np.array_equal(step.pool_image(l), G.expected_pool_image(w, store, l, FILL)), f"layer {l}"
