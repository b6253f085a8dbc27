"""The wrapper's one-expression checks pass only what its reporting checks pass (CPU tensors, no device)."""

import itertools

import pytest
import torch

import paper_2605_30842_amd.binding as B

CPU = torch.device("cpu")
BF, F32, I32 = torch.bfloat16, torch.float32, torch.int32
TENSORS = {
    "good": torch.zeros(3, 8, 64, dtype=BF),
    "float": torch.zeros(3, 8, 64),
    "transposed": torch.zeros(8, 3, 64, dtype=BF).transpose(0, 1),
    "short": torch.zeros(3, 8, 32, dtype=BF),
    "2-D": torch.zeros(24, 64, dtype=BF),
    "0-D": torch.zeros((), dtype=BF),
    "empty": torch.zeros(0, 8, 64, dtype=BF),
    "meta": torch.zeros(3, 8, 64, dtype=BF, device="meta"),
    "list": [1, 2, 3],
    "none": None,
}


def _passes(check, *args):
    try:
        check(*args)
        return True
    except ValueError:
        return False


@pytest.mark.parametrize("name", TENSORS)
def test_fits_implies_the_reported_check(name):
    t = TENSORS[name]
    for shape in ((3, 8, 64), (0, 8, 64), (3, 8, 32)):
        if B._fits(t, torch.Tensor, (BF,), CPU, shape):
            B._check_tensor("t", t, (BF,), CPU, shape=shape)
        else:
            assert not _passes(B._check_tensor, "t", t, (BF,), CPU, shape)


def _op():
    o = object.__new__(B.DecodeAttention)
    o.plan = None
    o.dtype = "bf16"
    o.num_q_heads, o.num_kv_heads, o.head_dim = 8, 2, 64
    o._torch_device = CPU
    o._q_dtypes, o._kv_dtypes = B._torch_dtypes("bf16")
    return o


def test_group_checks_agree_with_and_without_the_short_form(monkeypatch):
    """Each group check gives one verdict whether or not its short form is there to accept the call."""
    op = _op()
    out, lse = torch.zeros(3, 8, 64), torch.zeros(3, 8)
    kv = [torch.zeros(40, 2, 64, dtype=BF), torch.zeros(40, 4, 64, dtype=BF)[:, :2], torch.zeros(40, 2, 64),
          torch.zeros(4, 10, 2, 64, dtype=BF), torch.zeros(40, 2, 128, dtype=BF)[:, :, ::2], "k"]
    ints = [torch.zeros(3, dtype=I32), torch.zeros(3, dtype=torch.int64), torch.zeros(2, dtype=I32),
            torch.zeros(3, 4, dtype=I32), None]
    new = [torch.zeros(3, 2, 64, dtype=BF), torch.zeros(2, 2, 64, dtype=BF), torch.zeros(3, 2, 64)]
    calls = [(op._check_q_out, (q, o, x)) for q in TENSORS.values() for o in (out, None, out[:2]) for x in (lse, None)]
    calls += [(op._check_cache, (k, v, paged)) for k, v in itertools.product(kv, kv) for paged in (False, True)]
    calls += [(op._check_lengths, (c, 3, s, t)) for c, s, t in itertools.product(ints[:4], ints, ints)]
    calls += [(op._check_new_rows, (a, b, new[0], n)) for a, b in itertools.product(new, new) for n in (3, None)]
    calls += [(op._check_prefill, (q, s, n, 7, c, None, None, 64)) for q in list(TENSORS.values())[:4]
              for s, n, c in itertools.product(ints[:4], ints[:4], ints[:4])]
    short = [_passes(f, *a) for f, a in calls]
    monkeypatch.setattr(B, "_fits", lambda *a: False)
    assert [_passes(f, *a) for f, a in calls] == short
    assert any(short) and not all(short)


def test_prefill_without_scratch_when_it_cannot_be_had(monkeypatch):
    """Prefill scratch is an option: a full device or a foreign stream object leaves the call without it."""
    op = _op()
    monkeypatch.setattr(B, "comem_prefill_attn_workspace", lambda *a: 512)
    assert op._prefill_workspace(1, 40, 9000, None).numel() == 512
    assert op._prefill_workspace(1, 40, 9000, type("S", (), {"cuda_stream": 0})()) is None

    def full(*a, **kw):
        raise torch.OutOfMemoryError("full")

    monkeypatch.setattr(torch, "empty", full)
    assert op._prefill_workspace(1, 40, 9000, None) is None


def test_a_given_prefill_workspace_is_checked():
    op = _op()
    ws = torch.empty(512, dtype=torch.uint8)
    assert op._prefill_workspace(1, 40, 9000, None, ws) is ws
    for bad in (ws[::2], torch.empty(512, device="meta"), 512, [0]):
        with pytest.raises(ValueError):
            op._prefill_workspace(1, 40, 9000, None, bad)
