"""The cross-split merge and its tickets at the edges of their forms, against the oracle.

A lane of the merging workgroup takes one batch of at most 8 splits, or
batches of 16; 256 / (G * D / 4) lanes share an output slot (at least one).
Tickets lie 32 words apart, closer in plans of many sequences.
"""

import numpy as np
import pytest

import oracle.decode_attention as da
from tests.gpu_util import DeviceWorkload, check, make_op, run, say
from workloads.synth import WORKLOADS, generate, small_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,D", [(1, 64), (2, 64), (4, 128), (8, 128), (16, 128)])
@pytest.mark.parametrize("variant", ["mfma_grid", "valu"])
def test_split_counts_at_the_merge_batches(G, D, variant):
    lanes = max(1, 256 // (G * D // 4))
    counts = sorted({2, 8 * lanes - 1, 8 * lanes, 8 * lanes + 1, 16 * lanes, 16 * lanes + 1})
    lens = [32 * n - 5 for n in counts]
    spec = small_spec(WORKLOADS[2], lens, seed=400 + G).replace(num_q_heads=2 * G, num_kv_heads=2, head_dim=D)
    w = generate(spec)
    say(f"merge: G={G} D={D} {variant}, split counts {counts}")
    op = make_op(spec, chunk=32, variant=variant)
    dw = DeviceWorkload(w)
    ro, rl = da.reference(w)
    first = run(dw, op)
    check(*first, ro, rl, "bf16", f"G={G} D={D} {variant}")
    again = run(dw, op)  # the tickets are back at zero
    assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])


@pytest.mark.parametrize("max_batch", [63, 64, 128, 2046, 2047, 5000])
def test_ticket_spacing_of_large_plans(max_batch):
    """Plans whose tickets lie 32, 16, ... 1 words apart, called with debug checks: the error word and the
    queue counters lie past the last ticket."""
    lens = [700, 0, 1, 333]
    spec = small_spec(WORKLOADS[2], lens, seed=410)
    w = generate(spec)
    say(f"merge: tickets of a plan for {max_batch} sequences")
    op = make_op(spec, chunk=32, max_batch=max_batch, debug_checks=True)
    ro, rl = da.reference(w)
    for _ in range(2):
        check(*run(DeviceWorkload(w), op), ro, rl, "bf16", f"max_batch {max_batch}")
    assert op.device_errors() == 0
