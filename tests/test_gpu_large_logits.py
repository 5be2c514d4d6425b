"""bf16 attention where the logits' unit in the last place is many times the range of the exponential: a row is its largest
key's value, in every form of both matrix-core kernels.  The queries are multiplied by a power of two, so that the
oracle's rows are of the same inputs; no two largest logits of a row lie within the error of fp32 sums here."""
import numpy as np
import pytest

import mts_workloads as W
import oracle
from conftest import KERNEL_PREFILL, KERNEL_STREAMING
from helpers import as_values, draw_step_data
from test_gpu_parity import FILL, SCHEDULES, _harness, _oracle_store, check_attention
from test_gpu_prefill_split import SPLITS
from test_gpu_staged import _run as run_staged
from test_gpu_unappended import _run as run_unappended

pytestmark = pytest.mark.gpu

POWERS = [27, 33, 90]               # the largest scaled logits of a row: about 2^29, 2^35, 2^92
PREFIX, NEW = [700, 0, 333, 31, 1500], [20, 64, 33, 1, 47]


def _data(w, power):
    data = draw_step_data(w)
    for l in data["layers"]:
        data["q"][l] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(data["q"][l]) * np.float32(2.0) ** power)
    return data


def _check(w, power):
    data = _data(w, power)
    step = _harness().GpuStep(w, fill_byte=FILL)
    store = _oracle_store(w, data)
    step.unpack_histories(data, 0)
    step.append(data, 0)
    ref = oracle.attn_incremental(store, 0, data["q"][0], w.page_indptr, w.page_indices, w.prefix_lens, w.new_indptr)
    got = step.attention(data, 0)
    assert np.isfinite(as_values(got)).all()
    check_attention(w, got, ref)


@pytest.mark.parametrize("power", POWERS)
@pytest.mark.parametrize("schedule", list(SCHEDULES))
@pytest.mark.parametrize("D", [32, 64, 128])
def test_streaming(D, schedule, power, attn_tuning):
    attn_tuning(**{**SCHEDULES[schedule], "kernel": KERNEL_STREAMING})
    _check(W.custom_workload("huge", 40 + D, "bf16", 1, 2, D, 16, PREFIX, NEW, chunk_tokens=1024), power)


@pytest.mark.parametrize("power", POWERS)
@pytest.mark.parametrize("split", [None, *SPLITS])
@pytest.mark.parametrize("D", [64, 128])
def test_prefill(D, split, power, attn_tuning):
    attn_tuning(kernel=KERNEL_PREFILL, **(SPLITS[split] if split else {}))
    _check(W.custom_workload("huge", 50 + D, "bf16", 1, 2, D, 32, [1500, 0, 700, 33, 0], [8, 300, 0, 1, 127], chunk_tokens=1024), power)


@pytest.mark.parametrize("power", POWERS)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_rows_and_onload_buffer(D, power):
    w = W.custom_workload("huge", 60 + D, "bf16", 1, 2, D, 32, PREFIX, NEW, chunk_tokens=256)
    data = _data(w, power)
    run_unappended(w, data)
    run_staged(w, [0, 3], 256, data)
