"""States with many arcs under one label beside states with few.

A live state's arcs are shared out over lanes and threads; these FSTs put the
counts on both sides of where the sharing changes (16 arcs of an entry in a
workgroup, 256 arcs a round of a wavefront, 8 arcs of a lattice pair) and of
where a step goes to the streaming sweeps, and check both the results and that
no thread is left with a hub's arcs to itself (which made such passes tens to
thousands of times slower than the streaming sweeps).
"""
import numpy as np
import pytest

import synth
from gpu_common import assert_fb_parity, assert_final_parity, assert_viterbi_parity, say
from oracle import lattice as lat
from test_gpu_failed_calls import batch_of, bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


def skewed(Q, n, m, seed=0):
    """Label 0: start -> n states; label 1: each of them -> itself and a
    neighbour, and state 7 has m arcs more (parallel ones among them); label 2:
    all -> state 7."""
    rng = np.random.default_rng(seed)
    s = np.arange(1, n + 1)
    rows = np.concatenate([
        np.stack([0 * s, s, 0 * s], 1), np.stack([s, s, 0 * s + 1], 1), np.stack([s, 1 + s % n, 0 * s + 1], 1),
        np.stack([np.full(m, 7), rng.integers(1, n + 1, m), np.ones(m, int)], 1), np.stack([s, 0 * s + 7, 0 * s + 2], 1)])
    rows = rows[rng.permutation(len(rows))].astype(np.int32)
    a, b, c = (np.ascontiguousarray(rows[:, k]) for k in range(3))
    score = np.where(rng.random(len(rows)) < 0.2, -1.0, np.log(rng.uniform(0.05, 1.0, len(rows)))).astype(np.float32)
    return synth.Fst(Q, 3, 0, a, b, c, c.copy(), score, np.log(rng.uniform(0.1, 1.0, Q)).astype(np.float32))


STRINGS = [[0, 1], [0, 2, 1], [0, 1, 2, 1, 1], [0, 2, 1, 2, 1, 2, 1, 1], [0], [], [1], [0, 2, 2, 1]]


@pytest.mark.parametrize("Q,n,m", [(1203, 40, 200), (1203, 40, 257), (1203, 20, 513), (1203, 40, 1030), (1203, 9, 3000),
                                   (25011, 40, 2100), (25011, 40, 9000), (25011, 511, 16), (25011, 512, 17),
                                   (25011, 600, 500), (25011, 1030, 2100), (25011, 1030, 17), (25011, 1030, 5000)])
def test_parity(wf, Q, n, m):
    say(f"case: skewed Q={Q} n={n} m={m}")
    fst = skewed(Q, n, m, seed=n + m)
    d = wf.Fst.from_synth(fst)
    for copies in (1, 40):
        off, tok = batch_of(wf, copies, STRINGS)
        batch = synth.Batch(off.cpu().numpy().astype(np.int64), tok.cpu().numpy())
        ctx = f"skewed {Q} {n} {m} x{copies}"
        assert_viterbi_parity(fst, batch, d, ctx)
        assert_fb_parity(fst, batch, d, ctx)
        assert_final_parity(fst, batch, d, ctx)
        assert bits(wf.forward_backward(d, off, tok)) == bits(wf.forward_backward(d, off, tok))


@pytest.mark.parametrize("n,m", [(40, 8), (40, 9), (200, 400), (300, 2100), (300, 9000), (700, 30)])
def test_lattice_parity(wf, n, m):
    say(f"case: skewed lattice n={n} m={m}")
    fst = skewed(n + 3, n, m, seed=n + m)
    d = wf.Fst.from_synth(fst)
    w = lambda k: -0.1 * (k % 7)  # noqa: E731
    lattices = [(5, [(v, v + 1, lab, w(v + k)) for v, labs in enumerate([[0, 0], [2, 1], [1, 1, -1], [1, 2]])
                     for k, lab in enumerate(labs)]),
                (4, [(0, 1, 0, 0.0), (0, 2, 0, w(1)), (1, 2, 1, w(2)), (1, 3, 2, w(3)), (2, 3, 1, w(4))])]
    flat = wf.lattices_from_lists(lattices)
    lz, st, al = (x.cpu().numpy() for x in wf.lattice_forward(d, *flat, node_alpha=True))
    index = lat.label_index(fst)
    for b, (k, arcs) in enumerate(lattices):
        olz, A = lat.lattice_forward(fst, k, arcs, index=index)
        assert st[b] == wf.STATUS_OK and abs(float(lz[b]) - olz) <= 1e-4 * max(1.0, abs(olz))
        got = al[flat[0][b]:flat[0][b + 1]].astype(np.float64)
        fin = np.isfinite(A)
        assert np.array_equal(np.isfinite(got), fin)
        assert np.all(np.abs(got[fin] - A[fin]) <= 1e-4 * np.maximum(1.0, np.abs(A[fin])))
    assert d.health() == 0


def _time(f, runs=5):
    """Median milliseconds of a call."""
    import torch
    f()
    out = []
    for _ in range(runs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        out.append(a.elapsed_time(b))
    return sorted(out)[runs // 2]


def hub(Q, n, m):
    """Label 0: start -> n states, label 1: all -> hub, label 2: hub -> m arcs back."""
    s = np.arange(1, n + 1, dtype=np.int32)
    src = np.concatenate([0 * s, s, np.full(m, n + 1, np.int32)])
    dst = np.concatenate([s, 0 * s + n + 1, (1 + np.arange(m) % n).astype(np.int32)])
    lab = np.concatenate([0 * s, 0 * s + 1, np.full(m, 2, np.int32)])
    score = np.log(np.random.default_rng(m).uniform(0.1, 1, src.size)).astype(np.float32)
    return synth.Fst(Q, 3, 0, src, dst, lab, lab.copy(), score, np.zeros(Q, np.float32))


@pytest.mark.parametrize("Q,m", [(203, 1000), (25011, 3000), (25011, 16384)])
def test_hub_is_no_serial_chain(wf, Q, m):
    """Ten steps out of a hub: at most six times the streaming sweeps' time
    (it was 25 times for 1000 arcs and 600 times for 16384; now 1 to 2)."""
    say(f"case: hub time Q={Q} m={m}")
    fst = hub(Q, 40, m)
    off, tok = batch_of(wf, 16, [[0] + [1, 2] * 10])
    d, stream = wf.Fst.from_synth(fst), wf.Fst.from_synth(fst, state_memory=2)
    for name, call in (("viterbi", wf.viterbi), ("forward_backward", wf.forward_backward)):
        live, ref = _time(lambda: call(d, off, tok)), _time(lambda: call(stream, off, tok))
        say(f"  {name}: {live:.3f} ms, streaming {ref:.3f} ms")
        assert live <= 6 * ref, name


@pytest.mark.parametrize("m", [1000, 16384])
def test_lattice_hub_is_no_serial_chain(wf, m):
    """The same over a lattice (36 times and 300 times before)."""
    say(f"case: lattice hub time m={m}")
    fst = hub(203, 40, m)
    arcs = [(v, v + 1, 0 if v == 0 else 1 + (v + 1) % 2, -0.1 * k) for v in range(20) for k in range(2)]
    flat = wf.lattices_from_lists([(21, arcs)] * 16)
    d, stream = wf.Fst.from_synth(fst), wf.Fst.from_synth(fst, state_memory=2)
    live, ref = _time(lambda: wf.lattice_forward(d, *flat)), _time(lambda: wf.lattice_forward(stream, *flat))
    say(f"  {live:.3f} ms, streaming {ref:.3f} ms")
    assert live <= 6 * ref


def test_counts_of_left_sentences_by_slot(wf):
    """A string over 20000 of 25011 live states: its backward pass in the
    batch of left sentences takes at most 1.4 times the streaming form's time
    (1.7 times when it counted by (label, source) instead of by slot)."""
    say("case: counts of left sentences")
    rng = np.random.default_rng(1)
    Q, n, per = 25011, 20000, 10
    src = np.concatenate([np.zeros(n, int), np.repeat(np.arange(Q), per)]).astype(np.int32)
    dst = np.concatenate([np.arange(n), rng.integers(0, n, per * Q)]).astype(np.int32)
    lab = np.concatenate([np.zeros(n, int), np.ones(per * Q, int)]).astype(np.int32)
    o = np.lexsort((src, lab))
    fst = synth.Fst(Q, 2, 0, src[o], dst[o], lab[o], lab[o].copy(),
                    np.log(rng.uniform(0.1, 1, src.size)).astype(np.float32), np.zeros(Q, np.float32))
    off, tok = batch_of(wf, 2, [[0] + [1] * 12])
    ms = []
    for kw in ({}, {"state_memory": 2}):
        d = wf.Fst.from_synth(fst, **kw)
        wf.forward_backward(d, off, tok)
        d.profile(True)
        d.profile_read(reset=True)
        for _ in range(3):
            wf.forward_backward(d, off, tok)
        ms.append(d.profile_read()["backward"][0])
    say(f"  backward {ms[0]:.2f} ms, streaming {ms[1]:.2f} ms")
    assert ms[0] <= 1.4 * ms[1]
