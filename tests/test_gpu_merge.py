"""The cross-split merge and its tickets at the edges of their forms, against the oracle.

A lane of the merging workgroup takes one batch of at most 8 splits, or
batches of 16; 256 / (G * D / 4) lanes share an output slot (at least one).
Tickets lie 32 words apart, closer in calls of many sequences (of the plan's
most with a configured chunk).
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
@pytest.mark.parametrize("chunk", [32, 0])
def test_ticket_spacing_of_large_plans(max_batch, chunk):
    """Calls whose tickets lie 32, 16, ... 1 words apart, with debug checks: the error word and the queue counters
    lie before the first ticket."""
    lens = [700, 0, 1, 333]
    spec = small_spec(WORKLOADS[2], lens, seed=410)
    w = generate(spec)
    say(f"merge: tickets of a plan for {max_batch} sequences, chunk {chunk}")
    op = make_op(spec, chunk=chunk, max_batch=max_batch, debug_checks=True)
    ro, rl = da.reference(w)
    for _ in range(2):
        check(*run(DeviceWorkload(w), op), ro, rl, "bf16", f"max_batch {max_batch}")
    assert op.device_errors() == 0


@pytest.mark.parametrize("batch", [1, 3, 6, 12, 25, 50, 100, 200, 500])
def test_ticket_spacing_of_the_call(batch):
    """One plan and one workspace for 500 sequences, called with fewer and then with more: the spacing follows the
    call, and every call finds the tickets at zero."""
    lens = np.random.default_rng(420 + batch).integers(0, 200, size=batch).tolist()
    lens[0] = 199
    spec = small_spec(WORKLOADS[2], lens, seed=420).replace(num_q_heads=8, num_kv_heads=2, head_dim=64)
    w = generate(spec)
    say(f"merge: {batch} sequences of a plan for 500")
    op = make_op(spec, chunk=32, max_batch=500)
    ro, rl = da.reference(w)
    few = generate(small_spec(WORKLOADS[2], [199], seed=421).replace(num_q_heads=8, num_kv_heads=2, head_dim=64))
    few_ref = da.reference(few)
    for _ in range(2):
        check(*run(DeviceWorkload(w), op), ro, rl, "bf16", f"{batch} sequences")
        check(*run(DeviceWorkload(few), op), *few_ref, "bf16", "one sequence")


@pytest.mark.parametrize("ps,bound", [(1, 2016), (2, 4064)])
def test_whole_sequences_of_small_pages_without_a_workspace(ps, bound):
    """The longest sequence that runs whole in pages of 1 and 2 tokens, in a call that has no workspace."""
    spec = small_spec(WORKLOADS[4], [bound, 0, 31, bound - 1], max_ctx_len=bound, seed=450)
    spec = spec.replace(layout="paged", page_size=ps)
    w = generate(spec)
    op = make_op(spec, max_batch=64)
    op.workspace_bytes = 0
    say(f"merge: no workspace, page {ps}, {bound} tokens")
    check(*run(DeviceWorkload(w), op), *da.reference(w), "bf16", f"page {ps}")


def test_calls_of_a_small_workspace_agree_on_the_counters():
    """A long call over one-token pages whose partial results leave no room between tickets, then a call of eight
    short sequences that spread tickets would leave room for: it finds them at zero, not at the first one's
    results."""
    import torch

    spec = small_spec(WORKLOADS[4], [64000], max_ctx_len=64000, seed=440).replace(layout="paged", page_size=1)
    few = small_spec(WORKLOADS[2], [700, 650, 1, 700, 0, 699, 300, 700], max_ctx_len=700, seed=441)
    op = make_op(spec, max_batch=64)
    rows = 63 * spec.num_q_heads  # splits of 1024 tokens
    need = -(-(64 * spec.num_kv_heads + 3) * 4 // 256) * 256 + -(-rows * 4 // 256) * 256 + rows * spec.head_dim * 4
    op.workspace = torch.zeros(need, dtype=torch.uint8, device="cuda:0")
    op.workspace_bytes = need
    wl, ws = generate(spec), generate(few)
    rl, rs = da.reference(wl), da.reference(ws)
    say(f"merge: two calls in a workspace of {need} bytes")
    dl, ds = DeviceWorkload(wl), DeviceWorkload(ws)
    for _ in range(2):
        check(*run(dl, op), *rl, "bf16", "long")
        check(*run(ds, op), *rs, "bf16", "short")


@pytest.mark.parametrize("ps,chunk,bound", [(0, 64, 700), (16, 64, 700), (1, 0, 4000)])
def test_the_least_workspace(ps, chunk, bound):
    """The smallest workspace a call takes: dense counters and its partial results."""
    import torch

    lens = [700, 0, 1, 333] if chunk else [4000]
    spec = small_spec(WORKLOADS[4 if ps else 2], lens, max_ctx_len=bound, seed=430)
    spec = spec.replace(layout="paged", page_size=ps) if ps else spec
    w = generate(spec)
    op = make_op(spec, chunk=chunk, max_batch=64)
    splits = -(-bound // chunk) if chunk else 4  # planned: 1024 tokens
    rows = len(lens) * splits * spec.num_q_heads
    need = -(-(64 * spec.num_kv_heads + 3) * 4 // 256) * 256 + -(-rows * 4 // 256) * 256 + rows * spec.head_dim * 4
    say(f"merge: a workspace of {need} bytes, page {ps}, chunk {chunk}")
    op.workspace = torch.zeros(need, dtype=torch.uint8, device="cuda:0")
    op.workspace_bytes = need
    ro, rl = da.reference(w)
    first = run(DeviceWorkload(w), op)
    check(*first, ro, rl, "bf16", f"{need} bytes")
    again = run(DeviceWorkload(w), op)
    assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
    assert not op.workspace[:-(-(64 * spec.num_kv_heads + 3) * 4 // 256) * 256].any(), "counters back at zero"
