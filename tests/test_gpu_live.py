"""The live-state sweeps at the edges of their forms, against the oracle.

A fan FST puts n states live after its first symbol, so that n crosses the
list capacities (16 and 64 entries on chip, 512 for FSTs whose state vectors
exceed LDS, a quarter of the states in the global-memory form); a hub gives
one state m arcs under one label, so that m crosses the rounds of four arcs
per lane and the limits beyond which a sentence is left to the streaming
sweeps.  The three lookups of a label's arcs (the same number from every
state, a row per source, a hash table of pairs) each get an FST.  Viterbi
bit-exact; log Z within 1e-4 * max(1, |log Z|); posteriors within 1e-5 per
visit (the tolerances of the other sweeps).
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import assert_fb_parity, assert_final_parity, assert_viterbi_parity, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


def _fst(Q, M, arcs, seed, finals=0.8):
    """arcs: (src, dst, label) rows; random scores (ties among them), some states not final."""
    rng = np.random.default_rng(seed)
    a = np.asarray(arcs, np.int32)
    a = a[rng.permutation(len(a))]
    sc = np.where(rng.random(len(a)) < 0.2, -1.0, np.log(rng.uniform(0.05, 1.0, len(a)))).astype(np.float32)
    fin = np.where(rng.random(Q) < finals, np.log(rng.uniform(0.1, 1.0, Q)), -np.inf).astype(np.float32)
    return synth.Fst(Q, M, 0, a[:, 0].copy(), a[:, 1].copy(), a[:, 2].copy(), a[:, 2].copy(), sc, fin)


def _fan(Q, n, m, M=4, seed=0):
    """Label 0: start -> n states; label 1: each of them -> itself and its
    neighbour; label 2: all of them -> one hub, which has m arcs back to them
    (some of them parallel) under label 3."""
    s = np.arange(1, n + 1)
    rows = [(0, x, 0) for x in s]
    rows += [(x, x, 1) for x in s] + [(x, 1 + (x % n), 1) for x in s]
    rows += [(x, n + 1, 2) for x in s] + [(0, 0, 3)]
    rows += [(n + 1, 1 + (k * 7) % n, 3) for k in range(m)]
    return _fst(Q, M, rows, seed)


_STRINGS = [[0], [0, 1], [0, 1, 1, 1, 1], [0, 2], [0, 2, 3], [0, 1, 2, 3, 1, 2, 3, 1], [3, 3, 0, 1], [1], [], [2, 0],
            [0, 4], [3] * 9, [0, 2, 3, 2, 3, 2, 3, 1, 1, 1, 2]]


def _batch(copies=3):
    sents = _STRINGS * copies
    off = np.concatenate([[0], np.cumsum([len(s) for s in sents])]).astype(np.int64)
    return synth.Batch(off, np.concatenate([np.asarray(s, np.int32) for s in sents]))


def _check(fst, batch, d, ctx):
    assert_viterbi_parity(fst, batch, d, ctx)
    assert_fb_parity(fst, batch, d, ctx)
    assert_final_parity(fst, batch, d, ctx)


@pytest.mark.parametrize("n,m", [(1, 1), (3, 4), (15, 5), (16, 16), (17, 17), (63, 3), (64, 20), (65, 5), (200, 90)])
def test_fan(wf, n, m):
    say(f"case: fan n={n} m={m}")
    fst = _fan(n + 3, n, m, seed=n)
    _check(fst, _batch(), wf.Fst.from_synth(fst), f"fan {n} {m}")


@pytest.mark.parametrize("n,m,M", [(64, 3, 5), (511, 120, 5), (512, 130, 5), (513, 3, 600), (3000, 700, 600), (6000, 9, 5)])
def test_fan_wide(wf, n, m, M):
    """State vectors too large for LDS; M = 600 labels makes the pair table the lookup."""
    say(f"case: wide fan n={n} m={m} M={M}")
    fst = _fan(20011, n, m, M=M, seed=n)
    _check(fst, _batch(), wf.Fst.from_synth(fst), f"wide fan {n} {m} {M}")
    d = wf.Fst.from_synth(fst, checkpoint=1)
    assert_fb_parity(fst, _batch(), d, f"wide fan {n} {m} {M} checkpointed")


@pytest.mark.parametrize("tags,vocab", [(8, 20), (16, 50), (17, 50)])
def test_tagger_lookup(wf, tags, vocab):
    """The same number of arcs from every state under a label."""
    say(f"case: taggers {tags} tags")
    for fst, batch in (synth.config(4, n_tags=tags, vocab=vocab, batch=70, max_len=70),
                       synth.config(2, n_tags=tags, vocab=vocab, batch=70)):
        _check(fst, batch, wf.Fst.from_synth(fst), f"{tags} tags")


def test_left_sentences_by_option(wf):
    """Sentences left to the streaming sweeps: the same bits with the device
    list and as a batch of their own (forced checkpointing), whatever the
    count option, in a graph, and on repeats."""
    import torch
    fst = _fan(203, 200, 90, seed=3)
    batch = _batch(7)
    off = torch.as_tensor(batch.offsets.astype(np.int32), device="cuda")
    tok = torch.as_tensor(batch.tokens, device="cuda")
    got = []
    for kw in ({}, {}, {"checkpoint": 1}, {"count_records": -2}):
        say(f"case: left sentences {kw}")
        d = wf.Fst.from_synth(fst, **kw)
        for _ in range(2):
            s, a, st = wf.viterbi(d, off, tok)
            lz, post, fpost, st2 = wf.forward_backward(d, off, tok, final_posteriors=True)
            got.append([x.cpu().numpy().tobytes() for x in (s, a, st, lz, post, fpost, st2)])
            assert d.health() == 0
    d = wf.Fst.from_synth(fst)
    g = wf.Graph(d, off, tok, final=True)
    for _ in range(3):
        wf.viterbi(d, off, tok)
        g.replay()
        torch.cuda.synchronize()
        got.append([x.cpu().numpy().tobytes() for x in (g.best_score, g.best_arcs, g.status, g.log_z, g.grad,
                                                        g.grad_final, g.status)])
    g.close()
    for i, x in enumerate(got[1:]):
        assert x == got[0], f"run {i + 1} differs"


@pytest.mark.parametrize("n", [5, 40, 100])
def test_weighted_gradients_and_disabled_arcs(wf, n):
    """Scores of -inf written by set_scores disable arcs (as if they were not
    there); gradients under weights of both signs."""
    import torch
    say(f"case: disabled arcs n={n}")
    fst = _fan(n + 3, n, 30, seed=n)
    batch = _batch()
    off = np.random.default_rng(n).random(fst.num_arcs) < 0.3
    theta = fst.arc_score.copy()
    theta[off] = -np.inf
    keep = np.nonzero(~off)[0]
    sub = synth.Fst(fst.num_states, fst.num_ilabels, 0, fst.src[keep], fst.dst[keep], fst.ilabel[keep],
                    fst.olabel[keep], fst.arc_score[keep], fst.final_score)
    d = wf.Fst.from_synth(fst)
    th = torch.tensor(theta, device="cuda", requires_grad=True)
    lz, st = wf.log_partition(th, d, batch.offsets, batch.tokens)
    g = torch.linspace(-1.0, 2.0, batch.size, device="cuda") * (st == 0)
    (torch.where(st == 0, lz, torch.zeros_like(lz)) * g).sum().backward()
    olz, ograd, _, ost = oracle.forward_backward(sub, batch, grad_log_z=g.cpu().numpy().astype(np.float64))
    np.testing.assert_array_equal(st.cpu().numpy(), ost)
    ok = ost == oracle.ST_OK
    assert np.all(np.abs(lz.detach().cpu().numpy()[ok] - olz[ok]) <= 1e-4 * np.maximum(1, np.abs(olz[ok])))
    got = th.grad.cpu().numpy()
    n_k = np.bincount(batch.tokens, minlength=fst.num_ilabels + 1)[fst.ilabel]
    assert np.all(got[off] == 0)
    assert np.all(np.abs(got[keep] - ograd) <= 2e-5 * np.maximum(1, n_k[keep]))
    s, arcs, st = (x.cpu().numpy() for x in wf.viterbi(d, batch.offsets, batch.tokens))
    osc, oarcs, ost = oracle.viterbi(sub, batch)
    np.testing.assert_array_equal(st, ost)
    assert s.tobytes() == osc.tobytes()
    assert np.array_equal(arcs, np.where(oarcs >= 0, keep[oarcs], -1))
    assert d.health() == 0


def test_capture_after_eager(wf):
    """Viterbi and forward + backward captured by the caller after one eager call."""
    import torch
    fst = _fan(203, 200, 90, seed=4)
    batch = _batch(2)
    off = torch.as_tensor(batch.offsets.astype(np.int32), device="cuda")
    tok = torch.as_tensor(batch.tokens, device="cuda")
    d = wf.Fst.from_synth(fst)
    want = [x.clone() for x in wf.viterbi(d, off, tok)] + [x.clone() for x in wf.forward_backward(d, off, tok)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = list(wf.viterbi(d, off, tok)) + list(wf.forward_backward(d, off, tok))
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, want):
            assert x.cpu().numpy().tobytes() == y.cpu().numpy().tobytes()
        wf.viterbi(d, off, tok)
    assert d.health() == 0


@pytest.mark.parametrize("kind", ["fan", "tagger", "wide"])
def test_new_scores_reach_every_pass(wf, kind):
    """After set_scores every pass gives the bits of an FST created with the
    new scores: the sliced layouts' copies are rewritten by the first pass that
    reads them, eagerly, inside a library graph and inside the caller's
    capture, whichever pass comes first."""
    import torch
    say(f"case: new scores {kind}")
    if kind == "tagger":
        fst, batch = synth.config(4, n_tags=20, vocab=60, batch=40, max_len=30)
    else:
        fst, batch = _fan(20011 if kind == "wide" else 63, 60, 90, seed=5), _batch(2)
    rng = np.random.default_rng(7)
    off = torch.as_tensor(batch.offsets.astype(np.int32), device="cuda")
    tok = torch.as_tensor(batch.tokens, device="cuda")
    sents = [batch.sentence(b) for b in range(batch.size)]
    chain = wf.lattices_from_lists([(len(s) + 1, [(i, i + 1, int(a), -0.5) for i, a in enumerate(s)]) for s in sents])
    passes = {"viterbi": lambda d: wf.viterbi(d, off, tok), "fb": lambda d: wf.forward_backward(d, off, tok)}
    if kind != "wide":
        passes["noalloc"] = lambda d: wf.viterbi_noalloc(d, off, tok)
        passes["scan"] = lambda d: wf.forward_scan(d, off, tok, alpha=True)
        passes["lattice"] = lambda d: wf.lattice_forward(d, *chain)

    def bits(d, name):
        out = passes[name](d)
        torch.cuda.synchronize()
        return [x.cpu().numpy().tobytes() for x in out]

    d = wf.Fst.from_synth(fst)
    grouped = wf.Fst.from_synth(fst, count_records=-1)
    graph = wf.Graph(d, off, tok)
    names = list(passes)
    for step in range(len(names)):
        new = fst.arc_score + rng.normal(0, 0.3, fst.num_arcs).astype(np.float32)
        new[rng.integers(0, new.size)] = -0.0
        f2 = synth.Fst(**{**fst.__dict__})
        f2.arc_score = new
        ref, ref_grouped = wf.Fst.from_synth(f2), wf.Fst.from_synth(f2, count_records=-1)
        theta = torch.tensor(new, device="cuda")
        d.set_scores(theta)
        grouped.set_scores(theta)
        for name in names[step:] + names[:step]:
            assert bits(d, name) == bits(ref, name), f"{name} after set_scores"
        assert bits(grouped, "fb") == bits(ref_grouped, "fb")
        d.set_scores(torch.tensor(fst.arc_score, device="cuda"))
        d.set_scores(theta)
        graph.replay()
        torch.cuda.synchronize()
        want = [x.cpu().numpy().tobytes() for x in wf.viterbi(ref, off, tok)[:2]]
        assert [graph.best_score.cpu().numpy().tobytes(), graph.best_arcs.cpu().numpy().tobytes()] == want
        assert d.health() == 0
    graph.close()
    if kind != "wide":  # the update captured too
        theta = torch.tensor(fst.arc_score, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            d.set_scores(theta)
            out = passes["noalloc"](d)
        for _ in range(3):
            theta.add_(torch.as_tensor(rng.normal(0, 0.2, fst.num_arcs).astype(np.float32), device="cuda"))
            g.replay()
            torch.cuda.synchronize()
            f2 = synth.Fst(**{**fst.__dict__})
            f2.arc_score = theta.cpu().numpy()
            ref = wf.Fst.from_synth(f2)
            assert [x.cpu().numpy().tobytes() for x in out] == bits(ref, "viterbi")
            assert bits(d, "scan") == bits(ref, "scan")


@pytest.mark.parametrize("D,per,Q,M", [(1, 1, 3, 2), (3, 3, 9, 6), (8, 4, 11, 5), (8, 5, 11, 5), (9, 4, 20, 5), (16, 4, 16, 4),
                                       (16, 5, 30, 4), (17, 2, 30, 4), (5, 2, 20011, 600), (16, 3, 20011, 600)])
def test_narrow_labels(wf, D, per, Q, M):
    """At most D destinations per label and `per` parallel-or-not arcs of a
    label from one state: the edges of the 8- and 16-lane forms, every
    sentence length around their look-ahead, all lookups, paths that die."""
    say(f"case: narrow D={D} per={per} Q={Q} M={M}")
    rng = np.random.default_rng(100 * D + per)
    rows = []
    dests = [np.sort(rng.choice(min(Q, 40), D, replace=False)) for _ in range(M)]
    for a in range(M):
        for s in rng.choice(min(Q, 40), min(Q, 40) if a % 3 == 0 else max(1, min(Q, 40) // 2), replace=False):
            rows += [(s, d, a) for d in rng.choice(dests[a], rng.integers(0, per + 1))]
    rows += [(0, dests[0][k % D], 0) for k in range(per)]
    fst = _fst(Q, M, rows, D)
    lens = np.concatenate([np.arange(12), rng.integers(0, 40, 60), [130]])
    toks = rng.integers(0, min(M, 4), int(lens.sum())).astype(np.int32)
    toks[rng.random(toks.size) < 0.3] = 0
    toks[-3] = M  # a bad token
    batch = synth.Batch(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), toks)
    d = wf.Fst.from_synth(fst)
    _check(fst, batch, d, f"narrow {D} {per}")
    one = synth.Batch(np.array([0, 20], np.int64), toks[:20])
    _check(fst, one, d, f"narrow {D} {per} one sentence")


@pytest.mark.parametrize("n,m", [(3, 2), (40, 20), (383, 9), (384, 70), (385, 9), (600, 30), (1279, 9), (1290, 9)])
def test_lattice_lists(wf, n, m):
    """Lattice nodes whose live states cross the 384 and 1280 entries of its lists (larger
    ones are left to the streaming form), arcs that skip nodes, nodes with 64
    and 65 incoming arcs, pairs of one node above the workgroup's threads."""
    import torch
    from oracle import lattice as lat
    say(f"case: lattice lists n={n} m={m}")
    fst = _fan(n + 3, n, m, seed=n)
    w = lambda k: -0.1 * (k % 7)  # noqa: E731
    lattices = [
        (4, [(0, 1, 0, 0.0), (1, 2, 1, w(1)), (1, 2, -1, w(2)), (2, 3, 2, 0.0), (0, 3, 0, w(3)), (1, 3, -1, w(4))]),
        (3, [(0, 1, 0, w(1))] + [(1, 2, [1, 2, -1][k % 3], w(k)) for k in range(64)]),
        (3, [(0, 1, 0, w(1))] + [(1, 2, [1, 2, -1][k % 3], w(k)) for k in range(65)]),
        (2, [(0, 1, 1, 0.0)]),
        (6, [(0, 1, 0, 0.0), (1, 2, 2, w(1)), (2, 3, 3, w(2)), (1, 4, 1, w(3)), (3, 4, 1, w(4)), (0, 4, 3, w(5)),
             (4, 5, 1, w(6)), (3, 5, 2, w(1)), (2, 5, 3, w(2)), (0, 5, 0, w(3))]),
        (40, [(v, v + 1, [0, 1, 1, 2, 3][v % 5] if k < 2 else -1, w(v + k)) for v in range(39) for k in range(3)]),
        (1, []),
    ]
    d = wf.Fst.from_synth(fst)
    flat = wf.lattices_from_lists(lattices * 3)
    lz, st, al = (x.cpu().numpy() for x in wf.lattice_forward(d, *flat, node_alpha=True))
    lz2, st2 = (x.cpu().numpy() for x in wf.lattice_forward(d, *flat))
    torch.cuda.synchronize()
    assert d.health() == 0 and lz.tobytes() == lz2.tobytes() and st.tobytes() == st2.tobytes()
    index = lat.label_index(fst)
    for b, (k, arcs) in enumerate(lattices * 3):
        olz, A = lat.lattice_forward(fst, k, sorted(arcs, key=lambda e: e[1]), index=index)
        assert st[b] == (wf.STATUS_NO_PATH if olz == -np.inf else wf.STATUS_OK), b
        if olz != -np.inf:
            assert abs(float(lz[b]) - olz) <= 1e-4 * max(1.0, abs(olz)), b
        got = al[flat[0][b]:flat[0][b + 1]].astype(np.float64)
        fin = np.isfinite(A)
        np.testing.assert_array_equal(np.isfinite(got), fin, err_msg=f"lattice {b}")
        assert np.all(np.abs(got[fin] - A[fin]) <= 1e-4 * np.maximum(1.0, np.abs(A[fin]))), b


@pytest.mark.parametrize("D,per,lens", [
    (1, 1, [0, 1, 2, 15, 16, 17, 33, 200]), (8, 4, [255, 256, 257, 1, 0, 31, 32, 48, 512, 513]),
    (9, 4, [64, 65, 455, 456]), (16, 4, [1, 100, 256, 257, 300]), (0, 0, [1400, 700, 64, 65, 1370, 3])])
def test_scan_chunks(wf, D, per, lens):
    """The chunked one-launch scan: lengths on both sides of its 16 chunks and of
    its token window, bad tokens and offsets, log alpha of every token.  In FP64
    values with FP32 logarithms per step: 2e-7 a step, at most 1400 steps, so
    3e-4 absolute or 1e-6 relative."""
    import torch
    say(f"case: scan chunks D={D} per={per} lens={lens}")
    if D:
        rng = np.random.default_rng(D)
        dests = [np.sort(rng.choice(30, D, replace=False)) for _ in range(7)]
        fst = _fst(30, 7, [(s, d, a) for a in range(7) for s in range(0 if a != 3 else 14, 30)
                           for d in rng.choice(dests[a], rng.integers(1, per + 1))], D)
    else:
        fst = synth.config(4, n_tags=45, vocab=3000, batch=1, max_len=2)[0]
    d = wf.Fst.from_synth(fst)
    batch = synth.random_batch(3, fst.num_ilabels, lens + [5])
    toks = batch.tokens.copy()
    toks[-2] = fst.num_ilabels  # a bad token in the last sentence
    batch = synth.Batch(batch.offsets, toks)
    lz, st, al = (x.cpu().numpy() for x in wf.forward_scan(d, batch.offsets, batch.tokens, alpha=True))
    lz2, st2 = (x.cpu().numpy() for x in wf.forward_scan(d, batch.offsets, batch.tokens))
    torch.cuda.synchronize()
    assert lz.tobytes() == lz2.tobytes() and st.tobytes() == st2.tobytes()
    olz, _, _, ost = oracle.forward_backward(fst, batch, arc_posteriors=False)
    np.testing.assert_array_equal(st, ost)
    for b in range(batch.size):
        if ost[b] == oracle.ST_BAD_TOKEN:
            assert lz[b] == -np.inf
            continue
        want = oracle.fb_tables(fst, batch.sentence(b))[0][1:]
        got = al[batch.offsets[b]:batch.offsets[b + 1]].astype(np.float64)
        fin = np.isfinite(want)
        np.testing.assert_array_equal(np.isfinite(got), fin, err_msg=f"b={b}")
        assert np.all(np.abs(got[fin] - want[fin]) <= 3e-4 + 1e-6 * np.abs(want[fin])), b
        assert lz[b] == olz[b] or abs(lz[b] - olz[b]) <= 3e-4 + 1e-6 * abs(olz[b]), b


@pytest.mark.parametrize("Q,arcs,B", [(90, 500, 31), (90, 500, 32), (90, 9000, 70), (2600, 9000, 33), (6000, 4096, 40)])
def test_left_sentences_counted_by_label(wf, Q, arcs, B):
    """Sentences left to the streaming sweeps on both sides of the number from
    which their visits are counted by label: labels with more arcs and more
    visits than a workgroup takes, one, two and four visits staged at a time,
    bad tokens, empty sentences and paths that die among them."""
    say(f"case: left by label Q={Q} arcs={arcs} B={B}")
    rng = np.random.default_rng(Q + arcs + B)
    rows = [(0, d, 0) for d in range(1, 80)]  # more live states than a list holds
    for a in range(3):
        rows += list(zip(rng.integers(0, Q, arcs).tolist(), rng.integers(0, min(Q, 700), arcs).tolist(), [a] * arcs))
    rows += [(s, s, 3) for s in range(0, Q, 7)]
    fst = _fst(Q, 5, rows, Q)
    lens = rng.integers(1, 9, B)
    lens[5] = 0
    toks = rng.choice(4, int(lens.sum()), p=[0.5, 0.25, 0.15, 0.1]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    toks[off[:-1][lens > 0]] = 0
    toks[off[9] - 1] = 5 if lens[8] > 1 else 0  # a bad token
    toks[off[4] - 1] = 4                         # a label without arcs
    _check(fst, synth.Batch(off, toks), wf.Fst.from_synth(fst), f"left by label {Q} {arcs} {B}")


@pytest.mark.parametrize("tags,vocab,sents", [(3, 2, 7), (12, 60, 40), (45, 3000, 90)])
def test_counts_of_frequent_labels(wf, tags, vocab, sents):
    """A batch large enough for the backward sweep's cells of frequent labels
    (all labels, many of them, a few): a small batch repeated k times has k
    times its counts, whose sums differ by FP32 rounding (2^-24 each side) and
    fixed-point rounding (2^-31 a visit, scaled to the batch) only."""
    import torch
    say(f"case: frequent labels tags={tags} vocab={vocab}")
    rng = np.random.default_rng(tags)
    fst = synth.config(4, n_tags=tags, vocab=vocab, batch=1, max_len=2)[0]
    lens = rng.integers(0, 60, sents)
    toks = np.minimum(rng.geometric(0.15, int(lens.sum())) - 1, vocab - 1).astype(np.int32)
    if sents > 20:
        toks[-1] = vocab  # a bad token
    k = 300000 // int(lens.sum())
    w = rng.normal(0, 1, sents).astype(np.float32)
    d = wf.Fst.from_synth(fst)
    got = []
    for n in (1, k):
        off = np.concatenate([[0], np.cumsum(np.tile(lens, n))]).astype(np.int32)
        lz, st, tape = wf.forward(d, torch.as_tensor(off, device="cuda"), torch.as_tensor(np.tile(toks, n), device="cuda"))
        g, gf = wf.backward(d, tape, torch.as_tensor(np.tile(w, n), device="cuda"), final=True)
        torch.cuda.synchronize()
        tape.free()
        got.append([x.cpu().numpy().astype(np.float64) for x in (g, gf)])
    for one, many in zip(*got):
        assert np.any(one != 0)
        tol = k * (2.0 ** -23 * np.abs(one) + 2.0 ** -31 * lens.sum() * 4)
        assert np.all(np.abs(many - k * one) <= tol), np.max(np.abs(many - k * one) - tol)
    assert d.health() == 0


@pytest.mark.parametrize("n,m,copies", [(512, 2048, 3), (513, 2049, 3), (1024, 2047, 3), (2048, 30, 3), (2049, 3000, 3),
                                        (1025, 40, 3), (513, 600, 21), (2049, 5, 21)])
def test_workgroup_steps(wf, n, m, copies):
    """State vectors too large for LDS: lists and arcs of a step on both sides of
    what a workgroup keeps on chip (512 sources, 2048 arcs, 2048 destinations),
    with every sentence a workgroup's from the start (39 sentences) and only
    those a wavefront gave up (273)."""
    say(f"case: workgroup steps n={n} m={m} copies={copies}")
    fst = _fan(20011, n, m, seed=n + m)
    _check(fst, _batch(copies), wf.Fst.from_synth(fst), f"workgroup steps {n} {m} {copies}")
    small = _batch(1)
    _check(fst, small, wf.Fst.from_synth(fst), f"workgroup steps {n} {m}, touched list")
