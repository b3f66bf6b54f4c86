"""Accuracy of single steps and sums, each against the value it should have.

The tolerances are derived from the arithmetic that the header states, term by
term, not from measured results.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import say
from test_gpu_failed_calls import batch_of, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


def _final(wf, d, off, tok, w):
    import torch
    _, _, tape = wf.forward(d, off, tok)
    _, gf = wf.backward(d, tape, torch.as_tensor(w.astype(np.float32), device="cuda"), final=True)
    torch.cuda.synchronize()
    tape.free()
    return gf.cpu().numpy()


def _families():
    """Narrow labels, lists, sentences left to the streaming form, workgroup lists."""
    yield "narrow", synth.config(4, n_tags=9, vocab=40, batch=1, max_len=2)[0], [[k % 40, 3, 7 * k % 40] for k in range(50)] + [[]]
    yield "lists", fan(23, 20, 30, seed=2), None
    yield "left", fan(203, 200, 90, seed=3), None
    yield "workgroup", fan(25011, 900, 90, seed=4), None


def _case(wf, kind):
    for name, fst, strings in _families():
        if name == kind:
            return (fst,) + (batch_of(wf, 1, strings) if strings else batch_of(wf, 3))


@pytest.mark.parametrize("kind", ["narrow", "lists", "left", "workgroup"])
def test_final_posteriors_under_any_weight(wf, kind):
    """Weights scaled by a power of two scale the final-state posteriors
    exactly (every term is an FP32 product, their sum exact, one rounding), as
    long as no term is denormal; and a small weight's posteriors are as
    accurate as a large one's: an FP32 exponential of an argument whose FP32
    roundings are at most 2^-24 of 64 each (values up to 64 here, four of
    them), so 2^-16 relative."""
    say(f"case: final posteriors under any weight, {kind}")
    fst, off, tok = _case(wf, kind)
    d = wf.Fst.from_synth(fst)
    B = off.numel() - 1
    w = np.random.default_rng(1).normal(0, 1, B).astype(np.float32)
    base = _final(wf, d, off, tok, w)
    batch = synth.Batch(off.cpu().numpy().astype(np.int64), tok.cpu().numpy())
    assert np.any(base != 0)
    one = np.abs(w).astype(np.float64)
    want = oracle.forward_backward(fst, batch, grad_log_z=one, arc_posteriors=False, final_posteriors=True)[2]
    for k in (-60, -47, -20, 0, 60):
        got = _final(wf, d, off, tok, w * np.float32(2.0 ** k))
        keep = np.abs(base) > 2.0 ** -30
        assert np.array_equal(got[keep], (base[keep].astype(np.float64) * 2.0 ** k).astype(np.float32)), k
        got = _final(wf, d, off, tok, np.abs(w) * np.float32(2.0 ** k)).astype(np.float64) * 2.0 ** -k
        keep = want > 2.0 ** -30
        assert np.all(np.abs(got[keep] - want[keep]) <= 2.0 ** -16 * want[keep]), k
    assert d.health() == 0


@pytest.mark.parametrize("kind", ["narrow", "lists", "left"])
def test_final_posteriors_of_infinite_and_nan_weights(wf, kind):
    """An infinite weight makes the states its sentence can end in infinite, a
    NaN makes them NaN, and opposite infinities NaN; other states keep their sums."""
    say(f"case: infinite weights, {kind}")
    fst, off, tok = _case(wf, kind)
    d = wf.Fst.from_synth(fst)
    B = off.numel() - 1
    w = np.ones(B, np.float32)
    base = _final(wf, d, off, tok, w)
    reach = [_final(wf, d, off, tok, np.eye(B, dtype=np.float32)[b]) > 0 for b in (0, 1)]
    for v0, v1 in ((np.inf, 1.0), (-np.inf, 1.0), (np.nan, 1.0), (np.inf, -np.inf), (np.inf, np.inf)):
        w[:] = 1
        w[0], w[1] = v0, v1
        got = _final(wf, d, off, tok, w)
        with np.errstate(invalid="ignore"):
            want = np.where(reach[0], np.float32(v0), np.float32(0)) + np.where(reach[1] & ~np.isfinite(v1), np.float32(v1), np.float32(0))
        odd = ~np.isfinite(want)
        assert np.array_equal(got[odd], want[odd], equal_nan=True), (v0, v1)
        assert np.array_equal(got[~odd], base[~odd]), (v0, v1)
