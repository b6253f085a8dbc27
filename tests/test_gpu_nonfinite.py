"""Non-finite scores in decode, over every form a call can take and with one split and several: a NaN in K or q makes
the heads that see it NaN, output and lse; a score of -inf takes its token out of the softmax, also where it is all
that a tile, a wave or a whole split holds. Against the oracle."""

import numpy as np
import pytest

import oracle.decode_attention as da
from tests.gpu_util import TOL_DIAG, DeviceWorkload, make_op, run, say
from workloads.synth import WORKLOADS, generate, small_spec

pytestmark = pytest.mark.gpu

FORMS = {
    # name: base workload, lengths, length bound, plan's (chunk, variant), page size
    "one split": (2, [200, 31], 200, (0, "mfma_grid"), 0),
    "grid": (2, [700, 31], 700, (64, "mfma_grid"), 0),
    "strided, one split": (2, [90], 200, (0, "auto"), 0),
    "strided": (2, [3000], 3000, (0, "auto"), 0),
    "strided, page 4": (4, [3000], 3000, (0, "auto"), 4),
    "balanced": (2, [900, 0, 40, 2000], 131072, (0, "auto"), 0),
    "balanced, page 16": (4, [900, 0, 40, 2000], 131072, (0, "auto"), 16),
    "queue": (2, [6000, 31, 5000], 6000, (32, "auto"), 0),
    "fp8": (6, [3000], 3000, (0, "auto"), 0),
    "fp8, balanced, page 64": (7, [900, 0, 40, 2000], 131072, (0, "auto"), 64),
    "valu": (2, [90, 31], 90, (2048, "valu"), 0),
    "valu, several splits": (2, [700, 31], 700, (64, "valu"), 0),
    "valu f32": (1, [700, 31], 700, (64, "valu"), 0),
    "valu f32, page 2": (1, [700, 31], 700, (64, "valu"), 2),
}
NAN = {"bf16": np.uint16(0x7FC0), "f32": np.float32("nan"), "fp8": np.uint8(0x7F)}


def _draw(form, hq=8, hkv=2):
    base, lens, bound, (chunk, variant), ps = FORMS[form]
    spec = small_spec(WORKLOADS[base], lens, max_ctx_len=bound, seed=700 + len(form))
    spec = spec.replace(num_q_heads=hq, num_kv_heads=hkv, layout="paged" if ps else "contiguous", page_size=ps)
    return generate(spec), make_op(spec, chunk=chunk, variant=variant)


def _key(w, b, t):
    """Token t's K row [Hkv, D] of sequence b, as a view that can be written."""
    if w.spec.layout == "paged":
        ps = w.spec.page_size
        return w.k_pages[w.block_table[b, t // ps], t % ps]
    return w.k[w.seq_start[b] + t]


def _check(w, op, what):
    with np.errstate(invalid="ignore"):
        ref_out, ref_lse = da.reference(w)
    out, lse = run(DeviceWorkload(w), op)
    assert np.array_equal(np.isnan(lse), np.isnan(ref_lse)), f"{what}: heads with a NaN lse"
    assert np.array_equal(np.isnan(out), np.isnan(ref_out)), f"{what}: NaN outputs"
    fine = ~np.isnan(ref_lse)
    assert np.array_equal(np.isinf(lse[fine]), np.isinf(ref_lse[fine])), f"{what}: lse -inf"
    tol = TOL_DIAG * max(1.0, np.abs(ref_out[fine]).max(initial=0.0))
    assert np.abs(out[fine] - ref_out[fine]).max(initial=0.0) <= tol, what
    live = fine & np.isfinite(ref_lse)
    assert np.all(np.abs(lse[live] - ref_lse[live]) <= TOL_DIAG * np.maximum(1.0, np.abs(ref_lse[live]))), what
    return np.isnan(ref_lse)


@pytest.mark.parametrize("form", FORMS)
def test_a_nan_key_reaches_out_and_lse(form):
    """One NaN in one key of one KV head, at the first, an inner and the last token: its query heads are NaN."""
    for where in (0.0, 0.6, 1.0):
        w, op = _draw(form)
        t = int(where * (int(w.ctx_lens[0]) - 1))
        _key(w, 0, t)[1, 5] = NAN[w.spec.dtype]
        say(f"NaN key, {form}: token {t}")
        bad = _check(w, op, f"{form}, token {t}")
        assert bad[0, 4:].all() and bad.sum() == 4


@pytest.mark.parametrize("form", FORMS)
def test_a_nan_query_reaches_out_and_lse(form):
    """All scores of one query head NaN: no number comes out for it, and the others keep theirs."""
    w, op = _draw(form)
    w.q[0, 2, 7] = NAN[w.spec.q_dtype]
    say(f"NaN query, {form}")
    bad = _check(w, op, form)
    assert bad[0, 2] and bad.sum() == 1


@pytest.mark.parametrize("form", [f for f in FORMS if not f.startswith("fp8")])
@pytest.mark.parametrize("share", ["one", "first tile", "first half", "all but the last", "all"])
def test_a_score_of_minus_infinity_has_weight_zero(form, share):
    """Keys with an infinite component against the sign of q (one query head per KV head): scores of -inf."""
    w, op = _draw(form, hq=2, hkv=2)
    L = int(w.ctx_lens[0])
    n = {"one": 1, "first tile": 32, "first half": L // 2, "all but the last": L - 1, "all": L}[share]
    minus, plus = (np.uint16(0xFF80), np.uint16(0x7F80)) if w.spec.dtype == "bf16" else (np.float32("-inf"), np.float32("inf"))
    q0 = da.widen(w.q[0], w.spec.dtype)[1, 3]
    assert q0 != 0
    for t in range(min(n, L)):
        _key(w, 0, t)[1, 3] = minus if q0 > 0 else plus
    say(f"-inf scores, {form}: {share}")
    if share == "all":  # like an empty sequence: zeros and -inf (the definition's 0 / 0 has no value)
        out, lse = run(DeviceWorkload(w), op)
        assert np.all(out[0, 1] == 0) and lse[0, 1] == -np.inf and np.isfinite(lse[0, 0])
    else:
        _check(w, op, f"{form}, {share}")
