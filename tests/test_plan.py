"""Planning rules that need no GPU."""

import pytest

from paper_2605_30842_amd import binding as B
from tests.test_abi import _cfg, _contig_args, _noalloc_args, _paged_args


@pytest.mark.parametrize("max_batch", [1, 63, 64, 65, 127, 128, 1000, 2046, 2047, 2048, 4096])
def test_spread_tickets_fit_wherever_dense_ones_did(max_batch):
    """The allocation-free call takes a plan whose tickets and counters fit its 64 KiB counter region side by
    side, however far apart the plan then places them."""
    dense = -(-(max_batch * 8 + 3) * 4 // 256) * 256
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=max_batch, max_ctx_len=64), B.NO_DEVICE)
    try:
        st = B.load_library().comem_decode_attn_noalloc(*_noalloc_args(p, batch=1, max_ctx_len=64).values())
        assert st == (B.ERR_NO_DEVICE if dense <= 65536 else B.ERR_SCRATCH_LIMIT)
    finally:
        B.comem_decode_attn_destroy(p)


@pytest.mark.parametrize("batch,L,chunk", [
    (1, 100, 128),     # not worth a merge
    (1, 289, 320),
    (1, 290, 64),
    (16, 560, 576),    # two parts of a sequence save half of it
    (16, 561, 288),
    (1, 2048, 128),   # latency-bound: pieces worth their merge
    (1, 8192, 256),   # one split per compute unit
    (6, 4096, 832),   # 5 splits for each of 48 (sequence, head) pairs
    (4, 16384, 1024),  # never above 1024 while some unit is free
    (32, 1200, 1216),  # the pairs fill the chip: no split
    (32, 3000, 1024),  # one long sequence among short ones would run alone: ranges (splits without the workspace)
    (96, 1700, 1728),  # ... but not with several sequences to each range
])
def test_short_calls_plan_one_split_per_compute_unit(batch, L, chunk):
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=batch, max_ctx_len=L), B.NO_DEVICE)
    try:
        assert B.comem_decode_attn_plan_splits(p, batch, L, ws) == (chunk, -(-L // chunk))
    finally:
        B.comem_decode_attn_destroy(p)


def test_a_small_workspace_still_gets_every_call():
    """A workspace below what short splits need gets longer ones, down to one that needs none."""
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=1, max_ctx_len=8192), B.NO_DEVICE)
    try:
        sizes = [B.comem_decode_attn_plan_splits(p, 1, 8192, n)[0] for n in (ws, 600000, 300000, 40000, 0)]
        assert sizes == sorted(sizes) and sizes[0] == 256 and sizes[-1] >= 8192
    finally:
        B.comem_decode_attn_destroy(p)


def _dense(tickets):
    """Bytes of the counters with the tickets side by side."""
    return -(-(tickets + 3) * 4 // 256) * 256


def _partials(rows, d):
    return -(-rows * 4 // 256) * 256 + rows * d * 4


@pytest.mark.parametrize("max_batch", [1, 64, 511, 2047, 5000])
@pytest.mark.parametrize("variant", [B.VARIANT_AUTO, B.VARIANT_VALU])
def test_a_configured_chunk_needs_its_partial_results_and_dense_counters(max_batch, variant):
    """The least workspace that a call with chunk_tokens takes does not depend on how far apart tickets could lie."""
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=max_batch, max_ctx_len=640, chunk_tokens=64, variant=variant),
                                     B.NO_DEVICE)
    try:
        need = _dense(max_batch * 8) + _partials(max_batch * 10 * 32, 128)
        assert ws == need
        for n, status in ((need, B.ERR_NO_DEVICE), (need - 1, B.ERR_WORKSPACE_TOO_SMALL)):
            args = _contig_args(p, n, batch=max_batch, max_ctx_len=640)
            assert B.load_library().comem_decode_attn(*args.values()) == status
    finally:
        B.comem_decode_attn_destroy(p)


def test_debug_checks_need_room_for_dense_counters():
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=64, max_ctx_len=64, flags=B.FLAG_DEBUG_CHECKS), B.NO_DEVICE)
    try:
        for n, status in ((_dense(512), B.ERR_NO_DEVICE), (_dense(512) - 1, B.ERR_WORKSPACE_TOO_SMALL)):
            assert B.load_library().comem_decode_attn(*_contig_args(p, n, batch=1, max_ctx_len=64).values()) == status
    finally:
        B.comem_decode_attn_destroy(p)


@pytest.mark.parametrize("page,L", [(1, 2016), (2, 4064)])
def test_a_call_that_pages_allow_whole_needs_no_workspace(page, L):
    """A planned split spans at most 2046 pages; up to that length a sequence can run whole, whatever the plan
    prefers. One token more needs partial results."""
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=64, max_ctx_len=8192), B.NO_DEVICE)
    try:
        for n, status in ((L, B.ERR_NO_DEVICE), (L + 1, B.ERR_WORKSPACE_TOO_SMALL)):
            args = _paged_args(p, 0, batch=48, max_ctx_len=n, page_size=page, max_pages=n, workspace=None)
            assert B.load_library().comem_decode_attn_paged(*args.values()) == status
    finally:
        B.comem_decode_attn_destroy(p)


def test_one_token_pages_need_room_for_dense_counters():
    """A split of one-token pages has at most 2016 tokens (planned: 1024), so a long paged call needs some partial
    results."""
    p, ws = B.comem_decode_attn_init(_cfg(max_batch=64, max_ctx_len=4000), B.NO_DEVICE)
    try:
        need = _dense(512) + _partials(4 * 32, 128)
        for n, status in ((need, B.ERR_NO_DEVICE), (need - 1, B.ERR_WORKSPACE_TOO_SMALL)):
            args = _paged_args(p, n, batch=1, max_ctx_len=4000, page_size=1, max_pages=4000)
            assert B.load_library().comem_decode_attn_paged(*args.values()) == status
    finally:
        B.comem_decode_attn_destroy(p)


@pytest.mark.parametrize("kw,status", [
    (dict(), B.ERR_NO_DEVICE),
    (dict(workspace=None, workspace_bytes=0), B.ERR_NO_DEVICE),
    (dict(workspace=(1 << 20) + 16), B.ERR_MISALIGNED),
    (dict(q=None), B.ERR_NULL_POINTER),
    (dict(max_q_len=4097), B.ERR_INVALID_SHAPE),
    (dict(max_q_len=0, q=None), B.OK),
])
def test_prefill_split_validation(kw, status):
    from tests.test_abi import _prefill_args

    p, _ = B.comem_decode_attn_init(_cfg(), B.NO_DEVICE)
    try:
        args = _prefill_args(p)
        stream = args.pop("stream")
        args.update(workspace=1 << 20, workspace_bytes=1 << 20, stream=stream)
        args.update(kw)
        assert B.load_library().comem_prefill_attn_split(*args.values()) == status
    finally:
        B.comem_decode_attn_destroy(p)


def test_prefill_workspace_sizes():
    """A few new tokens over a long prefix use a workspace; a grid that fills the GPU, a short context and an
    empty call do not; a batch past the plan's is refused."""
    p, _ = B.comem_decode_attn_init(_cfg(max_batch=8, max_ctx_len=65536), B.NO_DEVICE)
    try:
        assert B.comem_prefill_attn_workspace(p, 1, 300, 24300) > 0
        for batch, m, L in ((1, 1024, 32768), (8, 2048, 65536), (1, 8192, 8192), (1, 300, 900), (0, 300, 24300),
                            (1, 0, 24300)):
            assert B.comem_prefill_attn_workspace(p, batch, m, L) == 0
        with pytest.raises(B.ComemError):
            B.comem_prefill_attn_workspace(p, 9, 300, 24300)
    finally:
        B.comem_decode_attn_destroy(p)


@pytest.mark.parametrize("hq,hkv,d,batch,m,L,splits", [
    (8, 4, 128, 1, 5000, 5000, False),   # causal: the blocks see half the keys on average
    (8, 4, 64, 1, 5000, 5000, False),
    (16, 8, 128, 2, 700, 12000, False),  # one round at two thirds of the units
    (16, 8, 64, 2, 700, 12000, True),    # ... whose shorter tiles a split evens out
    (32, 8, 64, 1, 300, 24300, True),
    (4, 4, 128, 1, 4000, 4000, True),    # causal, but half of the units idle
])
def test_prefill_splits_only_where_it_gains(hq, hkv, d, batch, m, L, splits):
    cfg = _cfg(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, max_batch=batch, max_ctx_len=L)
    p, _ = B.comem_decode_attn_init(cfg, B.NO_DEVICE)
    try:
        assert (B.comem_prefill_attn_workspace(p, batch, m, L) > 0) == splits
    finally:
        B.comem_decode_attn_destroy(p)
