"""The vector-ALU kernel at the edges of its tiles: every group size and row width, page sizes, and lengths around one
tile, one round of the four waves and one split, against the oracle."""

import numpy as np
import pytest

import oracle.decode_attention as da
from tests.gpu_util import DeviceWorkload, check, make_op, run, say
from workloads.synth import WORKLOADS, generate, small_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("ps", [0, 16, 2])
def test_tile_edges(dtype, d, group, ps):
    lens = [1, 7, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 255, 300, 0, 1025, 2047]
    spec = small_spec(WORKLOADS[1 if dtype == "f32" else 2], lens, seed=560 + group + ps)
    spec = spec.replace(num_q_heads=2 * group, num_kv_heads=2, head_dim=d)
    if ps:
        spec = spec.replace(layout="paged", page_size=ps)
    w = generate(spec, spare_pages=2, poison=True) if ps else generate(spec, gap_rows=3, poison=True)
    say(f"valu {dtype}, D {d}, G {group}, page {ps}")
    op, dw = make_op(spec, variant="valu"), DeviceWorkload(w)
    first = run(dw, op)
    check(*first, *da.reference(w), spec.dtype, f"G {group}")
    again = run(dw, op)
    assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
