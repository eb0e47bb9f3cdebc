"""extend_attention at the sizes where its kernels and dispatch rules change: edges of
the tiles and key steps, remainders, mixed batches.  Every row is checked against the
CPU oracle with LSE, over pools whose unused slots hold NaN."""

import numpy as np
import pytest

from paper_2609_32278_amd import workloads as wl
from test_gpu_extend import _run_and_compare

pytestmark = pytest.mark.gpu

NAN_FILL = {wl.KV_BF16: 0x7FC0, wl.KV_FP8_E4M3: 0x7F}

# prefixes whose last key falls on each edge of a 16-slot page, of a 64-key step and of
# the four waves' round of 256 keys; one long enough for many parts
STEP_EDGES = [0, 1, 14, 15, 16, 31, 47, 48, 62, 63, 64, 65, 127, 191, 254, 255, 256, 300, 2600]


@pytest.mark.parametrize("dt", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 128), (6, 2, 64), (16, 1, 64), (1, 1, 128)])
@pytest.mark.parametrize("split", [0, 64])
def test_decode_at_the_edges_of_pages_and_key_steps(dt, hq, hkv, d, split):
    w = wl.make_custom(STEP_EDGES, [1] * len(STEP_EDGES), hq, hkv, d, kv_dtype=dt, seed=61)
    _run_and_compare(w, f"decode_edges_{dt}_{hq}_{hkv}_{d}_{split}", want_lse=True, fill=NAN_FILL[dt],
                     split_keys=split)
