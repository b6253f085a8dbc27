"""Prefill calls whose keys several workgroups share, against the oracle: every split count up to the planned one, splits that a row or a whole block sees no key of, and the wrapper's own choice."""

import numpy as np
import pytest

import oracle.prefill_attention as pa
from tests.gpu_util import DevicePrefill, abs_values, check_prefill, make_op, run_prefill, say
from workloads.synth import PREFILL_WORKLOADS, generate_prefill, small_prefill_spec

pytestmark = pytest.mark.gpu


def _draw(ctx, new, ps, hq=32, hkv=8, d=128, seed=600):
    base = PREFILL_WORKLOADS[3 if ps else 1]
    spec = small_prefill_spec(base, ctx, new, seed=seed)
    kv = spec.kv.replace(num_q_heads=hq, num_kv_heads=hkv, head_dim=d)
    if ps:
        kv = kv.replace(page_size=ps)
    spec = spec.__class__(spec.name, kv, spec.new_tokens, spec.seed)
    return generate_prefill(spec, **(dict(spare_pages=2, poison=True) if ps else dict(gap_rows=3, poison=True)))


def _bytes(items, splits, d):
    rows = items * splits * 128
    return -(-rows * 4 // 256) * 256 + rows * d * 4


@pytest.mark.parametrize("ps,hq,hkv,d", [(0, 8, 2, 128), (16, 16, 2, 64), (1, 8, 2, 128), (64, 16, 1, 128), (0, 3, 3, 64)])
def test_every_split_count(ps, hq, hkv, d):
    """Sequences from all keys new (blocks that see only the first split) to a few over a long prefix, a
    partial last tile and an empty one, in one call; the workspace's size bounds the splits."""
    import torch

    import paper_2605_30842_amd.binding as B

    pw = _draw([2500, 700, 1024, 65, 0], [33, 130, 7, 65, 0], ps, hq, hkv, d, seed=601 + ps)
    dp = DevicePrefill(pw)
    kv = dp.kv
    s = pw.kv.spec
    op = make_op(s)
    blocks = -(-dp.max_q_len // (128 // s.group))
    items = s.batch * hkv * blocks
    want = pa.reference(pw)
    ref_abs = pa.reference(abs_values(pw))[0]
    planned = B.comem_prefill_attn_workspace(op.plan, s.batch, dp.max_q_len, s.max_ctx_len)
    say(f"prefill split: page {ps}, {hq}/{hkv} heads, D {d}, {items} items, planned {planned} bytes")
    most = next(n for n in range(2, 6) if _bytes(items, n, d) == planned)
    seen = []
    for splits in (1, 2, 3, 4, 5):
        nbytes = _bytes(items, splits, d) if splits > 1 else 0
        ws = torch.full((max(nbytes, 256),), 0xFF, dtype=torch.uint8, device="cuda:0")  # NaN partials
        out = torch.full(dp.q.shape, float("nan"), dtype=torch.float32, device="cuda:0")
        lse = torch.full(dp.q.shape[:2], float("nan"), dtype=torch.float32, device="cuda:0")
        head = (op.plan, dp.q.data_ptr(), dp.q_start.data_ptr(), dp.q_lens.data_ptr(), dp.max_q_len, kv.k.data_ptr(),
                kv.v.data_ptr())
        tail = (s.batch, s.max_ctx_len, out.data_ptr(), lse.data_ptr(), ws.data_ptr(), nbytes,
                torch.cuda.current_stream().cuda_stream)
        if ps:
            B.comem_prefill_attn_split_paged(*head, kv.k.stride(0), kv.k.stride(1), kv.k.stride(2), ps, kv.k.shape[0],
                                             kv.block_table.data_ptr(), kv.block_table.shape[1],
                                             kv.ctx_lens.data_ptr(), *tail)
        else:
            B.comem_prefill_attn_split(*head, kv.k.stride(0), kv.k.stride(1), kv.seq_start.data_ptr(),
                                       kv.ctx_lens.data_ptr(), *tail)
        torch.cuda.synchronize()
        out, lse = out.cpu().numpy(), lse.cpu().numpy()
        check_prefill(out, lse, *want, ref_abs, f"{splits} splits")
        seen.append(out)
    counts = len({o.tobytes() for o in seen})
    assert counts == most, f"{counts} different roundings from workspaces for 1 to {most} splits and more"


@pytest.mark.parametrize("ctx,new,ps", [([9000], [40], 0), ([9000, 3000], [100, 1], 16), ([8192], [8192], 0)])
def test_wrapper_splits_by_itself(ctx, new, ps):
    """The wrapper takes its own workspace (none where all tokens are new), on the current and on another stream, and
    repeats its bits."""
    import torch

    pw = _draw(ctx, new, ps, 8, 2, 128, seed=620)
    dp = DevicePrefill(pw)
    op = make_op(pw.kv.spec)
    say(f"prefill split wrapper: {ctx} {new} page {ps}")
    assert (op.prefill_workspace_bytes(len(ctx), max(new), max(ctx)) > 0) == (new != ctx)
    first = run_prefill(dp, op)
    rows = [(b, i, h) for b, m in enumerate(new) for i in {0, m // 2, m - 1} for h in (0, 7)]
    ref = pa.prefill_attention_rows(pw, rows)
    ref_abs = pa.prefill_attention_rows(abs_values(pw), rows)
    at = [(int(pw.q_start[b]) + i, h) for b, i, h in rows]
    check_prefill(np.stack([first[0][i, h] for i, h in at]), np.array([first[1][i, h] for i, h in at]),
                  np.stack([o for o, _ in ref]), np.array([x for _, x in ref]), np.stack([o for o, _ in ref_abs]),
                  "wrapper")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    kv, s = dp.kv, pw.kv.spec
    lse = torch.empty(dp.q.shape[:2], dtype=torch.float32, device="cuda:0")
    out = torch.empty(dp.q.shape, dtype=torch.float32, device="cuda:0")
    where = kv.block_table if ps else kv.seq_start
    call = op.prefill_paged if ps else op.prefill
    call(dp.q, dp.q_start, dp.q_lens, dp.max_q_len, kv.k, kv.v, where, kv.ctx_lens, s.max_ctx_len, out=out, lse=lse,
         stream=side)
    side.synchronize()
    assert np.array_equal(out.cpu().numpy(), first[0]) and np.array_equal(lse.cpu().numpy(), first[1])


def test_nan_key_reaches_out_and_lse():
    """A NaN key in one split's share makes the rows that see it NaN, outputs and lse, as in an unsplit call."""
    import torch

    pw = _draw([9000], [40], 0, 8, 2, 128, seed=630)
    dp = DevicePrefill(pw)
    kv, op = dp.kv, make_op(pw.kv.spec)
    say("prefill split: a NaN key")
    kv.k[int(pw.kv.seq_start[0]) + 4000, 1, 5] = float("nan")
    out, lse = (torch.from_numpy(x) for x in run_prefill(dp, op))
    assert out[:, 4:].isnan().all() and lse[:, 4:].isnan().all()
    assert out[:, :4].isfinite().all() and lse[:, :4].isfinite().all()


@pytest.mark.parametrize("keys", [1, 3000, 8000])
def test_keys_of_score_minus_infinity_in_the_first_splits(keys):
    """Rows whose first keys have scores of -inf, as many as several splits hold: those splits have weight 0."""
    pw = _draw([9000], [5], 0, 2, 2, 128, seed=640)
    t0 = int(pw.kv.seq_start[0])
    pw.q[:, 1, 7] = 0x3F80  # 1
    pw.kv.k[t0:t0 + keys, 1, 7] = 0xFF80  # -inf
    dp, op = DevicePrefill(pw), make_op(pw.kv.spec)
    splits = next(n for n in range(1, 65) if _bytes(2, n, 128) == op.prefill_workspace_bytes(1, 5, 9000))
    say(f"prefill split: {keys} keys of score -inf, {splits} splits")
    assert splits > 8, "the first batch of the merge holds 8"
    want = pa.reference(pw)
    check_prefill(*run_prefill(dp, op), *want, pa.reference(abs_values(pw))[0], f"{keys} keys")


def _call(dp, op, out, lse, ps, **kw):
    kv, s = dp.kv, dp.pw.kv.spec
    where = kv.block_table if ps else kv.seq_start
    (op.prefill_paged if ps else op.prefill)(dp.q, dp.q_start, dp.q_lens, dp.max_q_len, kv.k, kv.v, where, kv.ctx_lens,
                                             s.max_ctx_len, out=out, lse=lse, **kw)


@pytest.mark.parametrize("ps", [0, 16])
def test_a_given_workspace(ps):
    """A workspace of the reported size gives the bits of the wrapper's own scratch; an empty one the unsplit ones."""
    import torch

    pw = _draw([9000, 3000], [100, 1], ps, 8, 2, 128, seed=640)
    dp, op = DevicePrefill(pw), make_op(pw.kv.spec)
    say(f"prefill: a given workspace, page {ps}")
    want, want_lse = (torch.from_numpy(x) for x in run_prefill(dp, op))
    nbytes = op.prefill_workspace_bytes(2, dp.max_q_len, pw.kv.spec.max_ctx_len)
    assert nbytes > 0
    seen = []
    for n in (nbytes, 2 * nbytes, nbytes // 3, 0):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda:0")
        out, lse = torch.empty_like(want, device="cuda:0"), torch.empty_like(want_lse, device="cuda:0")
        _call(dp, op, out, lse, ps, workspace=ws)
        torch.cuda.synchronize()
        seen.append(out.cpu())
    assert torch.equal(seen[0], want) and torch.equal(seen[1], want)
    assert not torch.equal(seen[3], want) and torch.allclose(seen[3], want, atol=1e-4)
    assert torch.allclose(seen[2], want, atol=1e-4)


def test_captured_by_torch():
    """In a torch capture the scratch comes from the graph's pool: every replay gives the eager bits, whatever the
    program allocates and runs between them."""
    import torch

    pw = _draw([9000, 3000], [100, 1], 16, 8, 2, 128, seed=650)
    dp, op = DevicePrefill(pw), make_op(pw.kv.spec)
    say("prefill: captured by torch")
    want, want_lse = run_prefill(dp, op)
    out = torch.empty(want.shape, device="cuda:0")
    lse = torch.empty(want_lse.shape, device="cuda:0")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _call(dp, op, out, lse, 16)
        _call(dp, op, out, lse, 16)
    for i in range(4):
        out.zero_()
        junk = [torch.full((1 << 22,), 1e30 * i, device="cuda:0") for _ in range(8)]
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want) and np.array_equal(lse.cpu().numpy(), want_lse), f"replay {i}"
        del junk


def test_captured_by_another():
    """In a capture that torch did not begin the call keeps no scratch of torch's: it runs unsplit, and replays do
    not write to memory that other tensors have since got."""
    import ctypes

    import torch

    pw = _draw([9000, 3000], [100, 1], 0, 8, 2, 128, seed=660)
    dp, op = DevicePrefill(pw), make_op(pw.kv.spec)
    say("prefill: captured by another")
    want, want_lse = run_prefill(dp, op)
    unsplit = torch.empty(want.shape, device="cuda:0")
    lse = torch.empty(want_lse.shape, device="cuda:0")
    _call(dp, op, unsplit, lse, 0, workspace=torch.empty(0, dtype=torch.uint8, device="cuda:0"))
    torch.cuda.synchronize()
    out = torch.empty(want.shape, device="cuda:0")
    hip = ctypes.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream()
    raw, graph, ready = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(raw, 2) == 0  # relaxed
        _call(dp, op, out, lse, 0)
        assert hip.hipStreamEndCapture(raw, ctypes.byref(graph)) == 0
    assert hip.hipGraphInstantiate(ctypes.byref(ready), graph, None, None, 0) == 0
    with torch.cuda.stream(stream):
        held = [torch.full((1 << 20,), 7.0, device="cuda:0") for _ in range(64)]
    for i in range(3):
        stream.synchronize()
        out.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(ready, raw) == 0
        stream.synchronize()
        assert torch.equal(out, unsplit), f"replay {i}"
        assert all(bool((h == 7.0).all()) for h in held), f"replay {i}: another tensor's memory"
    assert hip.hipGraphExecDestroy(ready) == 0 and hip.hipGraphDestroy(graph) == 0
