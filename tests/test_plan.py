"""Planning rules that need no GPU."""

import pytest

from paper_2605_30842_amd import binding as B
from tests.test_abi import _cfg, _noalloc_args


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
