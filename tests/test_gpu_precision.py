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


@pytest.mark.parametrize("per", [1, 3, 40, 700])
def test_lattice_contributions_merge_in_fp64(wf, per):
    """Incoming arcs of a lattice node are log-added in FP64.  One state, a
    label with `per` arcs back to it, nodes joined by epsilon and labelled
    arcs whose weights add up to about 1: log Z stays near 0, where FP32 has
    digits to spare, so every merge shows.  Exact value in FP64; a node's
    error is its terms' roundings, 64 * 1280 * per terms of 2^-62 at most
    that many times each (the fixed point leaves room for that many), and the
    result's one FP32 rounding.  A labelled arc's own arcs may be summed in
    FP32 first (equal scores: 2^-22 with its logarithm), so those FSTs add
    that per node."""
    import torch
    say(f"case: lattice merges per={per}")
    z = np.zeros(per, np.int32)
    fst = synth.Fst(1, 1, 0, z, z, z, z, np.full(per, np.float32(-np.log(per) - 0.3)), np.zeros(1, np.float32))
    d = wf.Fst.from_synth(fst)
    rng = np.random.default_rng(per)
    worst = 0.0
    for nodes in (2, 30, 200):
        arcs, want = [], 0.0
        for v in range(nodes - 1):
            k = int(rng.integers(2, 6))
            p = rng.dirichlet(np.ones(k))
            w = np.log(p).astype(np.float32)
            arcs += [(v, v + 1, 0 if x % 2 else -1, float(w[x])) for x in range(k)]
            arc = np.log(per) + np.float64(fst.arc_score[0])
            t = np.array([w[x] + (arc if x % 2 else 0.0) for x in range(k)], np.float64)
            want += np.log(np.sum(np.exp(t)))
        lz, st = wf.lattice_forward(d, *wf.lattices_from_lists([(nodes, arcs)]))
        torch.cuda.synchronize()
        assert int(st[0]) == wf.STATUS_OK
        tol = nodes * (64 * 1280 * per) * 2.0 ** -62 * 6 * per + 2.0 ** -24 * abs(want) + 1e-13 * nodes
        err = abs(float(lz[0]) - want)
        worst = max(worst, err / tol)
        assert err <= tol, (nodes, err, tol)
    say(f"  worst error / tolerance {worst:.3g}")


@pytest.mark.parametrize("kw", [{}, {"checkpoint": 1}, {"state_memory": 2}])
@pytest.mark.parametrize("chunk", [11, 24, 37, 50])
def test_backward_chunks_add_no_rounding(wf, chunk, kw):
    """Backward values of a state whose arcs take several chunks.  Two branches
    of equal weight leave the start state; one fans out over 128 arcs of score
    0 and in again, 40 times, the other takes single arcs of score
    x = float(log 128).  The sum of a fan is the integer 128 in any chunking,
    so a level adds the FP32 logarithm's error only, 7 |fl(ln 2) - ln 2| =
    1.4e-8; the ratio of the branches' posteriors must be exp(40 (log 128 - x))
    up to that, and up to the posteriors' own roundings (exponentials of
    arguments below 1 formed by three FP32 additions, and the exponential and
    the result: 6 2^-24 each side)."""
    say(f"case: chunks of {chunk} arcs {kw}")
    K, m = 40, 128
    rows, n = [(0, 1, 0), (0, 2, 0)], 3
    a, b, scores = 1, 2, [0.0, 0.0]
    x = np.float32(np.log(m))
    for _ in range(K):
        mid = list(range(n, n + m))
        b1, a2, b2 = n + m, n + m + 1, n + m + 2
        n += m + 3
        rows += [(a, d, 1) for d in mid] + [(b, b1, 1)] + [(d, a2, 2) for d in mid] + [(b1, b2, 2)]
        scores += [0.0] * m + [x] + [0.0] * m + [0.0]
        a, b = a2, b2
    r = np.asarray(rows, np.int32)
    fst = synth.Fst(n, 3, 0, r[:, 0].copy(), r[:, 1].copy(), r[:, 2].copy(), r[:, 2].copy(),
                    np.asarray(scores, np.float32), np.zeros(n, np.float32))
    d = wf.Fst.from_synth(fst, chunk_arcs=chunk, **kw)
    off, tok = batch_of(wf, 1, [[0] + [1, 2] * K])
    _, post, st = wf.forward_backward(d, off, tok)
    p = post.cpu().numpy().astype(np.float64)
    assert int(st[0]) == wf.STATUS_OK and d.health() == 0
    got, want = np.log(p[0] / p[1]), K * (np.log(np.float64(m)) - np.float64(x))
    assert abs(got - want) <= K * 1.4e-8 + 12 * 2.0 ** -24, (got, want)


@pytest.mark.parametrize("n,copies", [(2000, 1), (6000, 1), (6000, 300)])
def test_small_terms_round_to_nearest(wf, n, copies):
    """Terms far below a sum's largest: a loop of score 0 beside n parallel
    loops of 1.9 2^-31 of it each.  A term is a fixed-point number of unit
    2^-31 rounded to nearest, so a step of log Z is off by at most n 2^-32,
    plus the exponentials' own error (arguments of -21: 2^-18 relative) and two
    FP32 roundings near 1 with its logarithm's (2^-22 together)."""
    say(f"case: small terms n={n} copies={copies}")
    Q, T = 25011, 9
    y = np.float32(np.log(1.9 * 2.0 ** -31))
    one = np.ones(n + 1, np.int32)
    src = np.concatenate([[0], one, [3]]).astype(np.int32)
    dst = np.concatenate([[1], one, [4]]).astype(np.int32)
    lab = np.concatenate([[0], one, [2]]).astype(np.int32)
    score = np.concatenate([[0.0, 0.0], np.full(n, y), [0.0]]).astype(np.float32)
    d = wf.Fst(Q, 3, 0, src, dst, lab, score, np.zeros(Q, np.float32))
    off, tok = batch_of(wf, copies, [[0] + [1] * T])
    lz, st, tape = wf.forward(d, off, tok)
    lz = lz.cpu().numpy().astype(np.float64)
    tape.free()
    small = n * np.exp(np.float64(y))
    err = np.abs(lz - T * np.log1p(small))
    assert np.all(err <= T * (n * 2.0 ** -32 + small * 2.0 ** -18 + 2.0 ** -22)), err.max()
    assert d.health() == 0
