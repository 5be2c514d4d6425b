"""Large calls of long users load their K/V tiles past the caches: the same arithmetic on the same
schedule, so the same bits as ordinary loads.  The form is chosen by the call's page count
(kv_past_caches); here a small batch states a large one."""
import numpy as np
import pytest

import mts_workloads as W
from conftest import KERNEL_STREAMING
from helpers import draw_step_data
from test_gpu_parity import FILL, _harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,S", [(32, 16), (64, 32), (128, 16)])
@pytest.mark.parametrize("new", [5, 20, 40, 64])
def test_tiles_loaded_past_the_caches_give_the_same_bits(D, S, new, attn_tuning):
    attn_tuning(kernel=KERNEL_STREAMING, min_tiles=2)
    G = _harness()
    w = W.custom_workload("past_caches", 40 + D + new, "bf16", 1, 3, D, S, [0, 31, 700, 1290], [new, 1, new, new - 1],
                          chunk_tokens=256)
    data = draw_step_data(w)
    step = G.GpuStep(w, fill_byte=FILL)
    step.unpack_histories(data, 0)
    step.append(data, 0)

    def outputs():
        return [step.attention(data, 0), step.attention_pointwise(data, 0, 0.01), step.attention_unappended(data, 0),
                step.attention_unappended(data, 0, inv_norm=0.01)]

    plain = outputs()
    meta = step.batch.meta
    meta.total_pages = (400 << 20) // step.cache.page_bytes + 1
    for a, b in zip(plain, outputs()):
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
