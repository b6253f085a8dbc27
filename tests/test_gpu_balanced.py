"""The balanced form (equal ranges of all sequences' tokens) at the edges of its geometry, against the oracle.

Planned calls take it when their length bound is long enough; here the bound is far above most lengths, so that
ranges are short, hold several sequences, end inside and between them, and some stay empty.
"""

import numpy as np
import pytest

import oracle.decode_attention as da
from tests.gpu_util import DeviceWorkload, check, make_op, run, say, to_torch
from workloads.synth import WORKLOADS, draw_new_rows, generate, small_spec

pytestmark = pytest.mark.gpu


def _spec(base, lens, bound, ps=0, **heads):
    spec = small_spec(WORKLOADS[base], lens, max_ctx_len=bound, seed=500 + len(lens) + ps)
    spec = spec.replace(**heads) if heads else spec
    return spec.replace(layout="paged", page_size=ps) if ps else spec.replace(layout="contiguous", page_size=0)


def _ragged(batch, top, seed):
    r = np.random.default_rng(seed)
    lens = r.integers(0, top, batch)
    edge = [0, 1, 32, 33, 2048, 2047, 0, 64]
    lens[:min(batch, 8)] = edge[:min(batch, 8)]
    return lens.tolist()


CASES = {
    # name: base workload, lengths, bound, page size, head counts
    "one long": (2, [40000], 40000, 0, {}),
    "bound far above the length": (2, [77], 131072, 0, {}),
    "two equal": (2, [8192, 8192], 262144, 0, {}),
    "empty between": (2, [5000, 0, 0, 3, 7000], 131072, 0, {}),
    "all empty": (2, [0, 0, 0], 131072, 0, {}),
    "64 sequences": (2, _ragged(64, 3000, 1), 8192, 0, {}),
    "65 sequences (offsets in LDS)": (2, _ragged(65, 3000, 2), 8192, 0, {}),
    "page 16": (4, _ragged(9, 9000, 3), 65536, 16, {}),
    "page 128": (4, _ragged(9, 9000, 4), 65536, 128, {}),
    "page 8": (4, _ragged(7, 5000, 5), 65536, 8, {}),
    "page 1": (4, _ragged(7, 5000, 6), 65536, 1, {}),
    "fp8": (6, _ragged(9, 9000, 7), 65536, 0, {}),
    "fp8 page 64": (7, _ragged(9, 9000, 8), 65536, 64, {}),
    "fp8 page 1": (7, _ragged(5, 3000, 9), 65536, 1, {}),
    "5 heads, D 64": (2, _ragged(9, 9000, 10), 65536, 0, dict(num_q_heads=10, num_kv_heads=5, head_dim=64)),
    "G 16": (2, _ragged(9, 9000, 11), 65536, 0, dict(num_q_heads=32, num_kv_heads=2)),
    "40 heads": (2, _ragged(9, 2500, 12), 65536, 16, dict(num_q_heads=40, num_kv_heads=40, head_dim=64)),
    "43 heads (two ranges a unit)": (2, _ragged(9, 2500, 13), 65536, 0, dict(num_q_heads=43, num_kv_heads=43, head_dim=64)),
    "64 heads": (2, _ragged(5, 2500, 14), 65536, 0, dict(num_q_heads=64, num_kv_heads=64, head_dim=64)),
    "65 heads (splits)": (2, _ragged(5, 2500, 15), 65536, 0, dict(num_q_heads=65, num_kv_heads=65, head_dim=64)),
    "one long, 128 heads": (2, [4001], 4001, 0, dict(num_q_heads=128, num_kv_heads=128, head_dim=64)),
    "one long, 129 heads (splits)": (2, [4001], 4001, 0, dict(num_q_heads=129, num_kv_heads=129, head_dim=64)),
    "more splits than workgroups": (6, [8192, 3000], 8192, 0, dict(num_q_heads=66, num_kv_heads=66, head_dim=64)),
    "600 heads (no split)": (2, [700, 0, 33], 65536, 0, dict(num_q_heads=600, num_kv_heads=600, head_dim=64)),
}


@pytest.mark.parametrize("name", CASES)
def test_balanced_matches_the_oracle(name):
    base, lens, bound, ps, heads = CASES[name]
    spec = _spec(base, lens, bound, ps, **heads)
    w = generate(spec, spare_pages=2, poison=True) if ps else generate(spec, gap_rows=5, poison=True)
    say(f"balanced {name}: batch {len(lens)}, {spec.dtype}, page {ps}")
    op, dw = make_op(spec), DeviceWorkload(w)
    first = run(dw, op)
    ro, rl = da.reference(w)
    check(*first, ro, rl, spec.dtype, name)
    again = run(dw, op)
    assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])


def test_balanced_at_the_batch_limit():
    lens = np.random.default_rng(520).integers(0, 65, size=4096).tolist()
    spec = _spec(2, lens, 4096, num_q_heads=8, num_kv_heads=2, head_dim=64)
    w = generate(spec)
    say("balanced: 4096 sequences")
    ro, rl = da.reference(w)
    check(*run(DeviceWorkload(w), make_op(spec)), ro, rl, spec.dtype, "4096 sequences")


@pytest.mark.parametrize("base,ps", [(2, 0), (4, 16), (4, 1), (7, 64)])
def test_balanced_fused_append(base, ps):
    """Store-and-attend in one launch leaves the cache and output bits of the two calls."""
    import torch

    lens = [max(1, n) for n in _ragged(9, 9000, 21)]
    spec = _spec(base, lens, 65536, ps)
    w = generate(spec, spare_pages=2) if ps else generate(spec)
    nk, nv = draw_new_rows(spec, seed=521)
    tk, tv = to_torch(nk, spec.dtype, "cuda:0"), to_torch(nv, spec.dtype, "cuda:0")
    a, b = DeviceWorkload(w), DeviceWorkload(w)
    op = make_op(spec)
    say(f"balanced fused append: {spec.dtype}, page {ps}")
    if ps:
        op.append_paged(tk, tv, a.k, a.v, a.block_table, a.ctx_lens, spec.max_ctx_len)
        out_a, _ = op.forward_paged(a.q, a.k, a.v, a.block_table, a.ctx_lens, spec.max_ctx_len)
        out_b, _ = op.append_forward_paged(b.q, tk, tv, b.k, b.v, b.block_table, b.ctx_lens, spec.max_ctx_len)
    else:
        op.append(tk, tv, a.k, a.v, a.seq_start, a.ctx_lens, spec.max_ctx_len)
        out_a, _ = op.forward(a.q, a.k, a.v, a.seq_start, a.ctx_lens, spec.max_ctx_len)
        out_b, _ = op.append_forward(b.q, tk, tv, b.k, b.v, b.seq_start, b.ctx_lens, spec.max_ctx_len)
    torch.cuda.synchronize()
    assert torch.equal(a.k, b.k) and torch.equal(a.v, b.v) and torch.equal(out_a, out_b)


@pytest.mark.parametrize("base,ps", [(2, 0), (4, 16), (4, 1), (6, 0), (7, 64)])
@pytest.mark.parametrize("length", [1, 31, 32, 33, 64, 65, 257, 288, 289, 321, 448, 449, 641, 2049, 6001])
def test_one_sequence_in_strided_tiles(base, ps, length):
    """One sequence: every split takes every n-th tile; the last tile, whichever split and wave has it, is partial and
    takes the fused append's row."""
    import torch

    spec = _spec(base, [length], 8192, ps)
    w = generate(spec, spare_pages=2, poison=True) if ps else generate(spec, gap_rows=5, poison=True)
    nk, nv = draw_new_rows(spec, seed=540 + length)
    tk, tv = to_torch(nk, spec.dtype, "cuda:0"), to_torch(nv, spec.dtype, "cuda:0")
    a, op = DeviceWorkload(w), make_op(spec)
    say(f"strided tiles: {length} tokens, {spec.dtype}, page {ps}")
    ro, rl = da.reference(w)
    check(*run(a, op), ro, rl, spec.dtype, f"{length} tokens")
    b = DeviceWorkload(w)
    where_a, where_b = (a.block_table, b.block_table) if ps else (a.seq_start, b.seq_start)
    (op.append_paged if ps else op.append)(tk, tv, a.k, a.v, where_a, a.ctx_lens, spec.max_ctx_len)
    out_a, _ = (op.forward_paged if ps else op.forward)(a.q, a.k, a.v, where_a, a.ctx_lens, spec.max_ctx_len)
    fused = op.append_forward_paged if ps else op.append_forward
    out_b, _ = fused(b.q, tk, tv, b.k, b.v, where_b, b.ctx_lens, spec.max_ctx_len)
    torch.cuda.synchronize()
    same = lambda x, y: torch.equal(x.view(torch.uint8), y.view(torch.uint8))  # noqa: E731 (NaN poison compares as bytes)
    assert same(a.k, b.k) and same(a.v, b.v) and torch.equal(out_a, out_b)


@pytest.mark.parametrize("chunk,variant", [(256, "auto"), (0, "mfma_grid"), (0, "valu")])
def test_forms_without_ranges_do_not_see_the_neighbours(chunk, variant):
    """A sequence's bits stay the same whatever the other sequences' lengths are."""
    import dataclasses

    lens = _ragged(9, 5000, 31)
    w = generate(_spec(2, lens, 16384))
    op = make_op(w.spec, chunk=chunk, variant=variant)
    say(f"neighbours: chunk {chunk}, {variant}")
    out, lse = run(DeviceWorkload(w), op)
    other = np.array([n if b % 2 else max(1, n // 3) for b, n in enumerate(lens)])
    out2, lse2 = run(DeviceWorkload(dataclasses.replace(w, ctx_lens=other)), op)
    assert np.array_equal(out[1::2], out2[1::2]) and np.array_equal(lse[1::2], lse2[1::2])
