"""Calls that fail, and the calls after them.

A call that runs out of memory in its middle must leave nothing behind that a
later call reads: the next call on the same FST gives the bits a fresh FST
gives.  Allocation failures are forced from the host (debug_alloc_limit: the
library refuses the allocation before asking the device), so every kernel
queued before the failure runs and ends normally.
"""
import numpy as np
import pytest

import synth
from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


def fan(Q, n, m, seed=0, M=4):
    """Label 0: start -> n states; label 1: each of them -> itself and its
    neighbour; label 2: all -> one hub, whose m arcs under label 3 lead back."""
    rng = np.random.default_rng(seed)
    s = np.arange(1, n + 1)
    rows = np.concatenate([
        np.stack([0 * s, s, 0 * s], 1), np.stack([s, s, 0 * s + 1], 1), np.stack([s, 1 + s % n, 0 * s + 1], 1),
        np.stack([s, 0 * s + n + 1, 0 * s + 2], 1), [[0, 0, 3]],
        np.stack([np.full(m, n + 1), 1 + (np.arange(m) * 7) % n, np.full(m, 3)], 1)]).astype(np.int32)
    rows = rows[rng.permutation(len(rows))]
    a, b, c = (np.ascontiguousarray(rows[:, k]) for k in range(3))
    score = np.log(rng.uniform(0.05, 1.0, len(rows))).astype(np.float32)
    return synth.Fst(Q, M, 0, a, b, c, c.copy(), score, np.log(rng.uniform(0.1, 1.0, Q)).astype(np.float32))


STRINGS = [[0], [0, 1, 1, 1, 1], [0, 2, 3], [0, 1, 2, 3, 1, 2, 3, 1], [3, 3, 0, 1], [], [3] * 9, [0, 2, 3, 2, 3, 1, 1, 2]]


def batch_of(wf, copies, strings=STRINGS):
    off, tok = wf.batch_from_sentences(strings * copies)
    import torch
    return torch.as_tensor(off, device="cuda"), torch.as_tensor(tok, device="cuda")


def bits(xs):
    import torch
    torch.cuda.synchronize()
    return [x.cpu().numpy().tobytes() for x in xs]


@pytest.mark.parametrize("kw", [{"checkpoint": 1}, {"checkpoint": 1, "count_records": -2}])
def test_backward_after_a_failed_backward(wf, kw):
    """A backward pass that fails after its first counts (no room for the
    buffers of the sentences left to the streaming sweeps), then others."""
    say(f"case: failed backward {kw}")
    fst = fan(203, 200, 90, seed=1)
    small, large = batch_of(wf, 1), batch_of(wf, 40)
    want = bits(wf.forward_backward(wf.Fst.from_synth(fst, **kw), *small, final_posteriors=True))
    d = wf.Fst.from_synth(fst, **kw)
    assert bits(wf.forward_backward(d, *small, final_posteriors=True)) == want
    for _ in range(2):
        _, _, tape = wf.forward(d, *large)
        d.debug_alloc_limit(1)
        with pytest.raises(wf.WfstError) as e:
            wf.backward(d, tape, final=True)
        assert e.value.code == wf.WFST_ENOMEM
        d.debug_alloc_limit(0)
        tape.free()
        assert bits(wf.forward_backward(d, *small, final_posteriors=True)) == want
    full = bits(wf.forward_backward(d, *large, final_posteriors=True))
    assert full == bits(wf.forward_backward(wf.Fst.from_synth(fst, **kw), *large, final_posteriors=True))
    assert d.health() == 0


def test_backward_state_memory_lds_only(wf):
    """state_memory=1 refuses a backward pass whose streaming form does not
    fit LDS, whatever the size of the batch and the live states of its
    sentences (forward: 12000 states and 5000 destinations fit)."""
    say("case: state_memory=1, backward beyond LDS")
    Q, D = 12000, 5000
    s = np.arange(D, dtype=np.int32)
    src = np.concatenate([s, [0]]).astype(np.int32)
    dst = np.concatenate([s, [1]]).astype(np.int32)
    lab = np.concatenate([0 * s, [1]]).astype(np.int32)
    d = wf.Fst(Q, 2, 0, src, dst, lab, np.full(src.size, -0.5, np.float32), np.zeros(Q, np.float32), state_memory=1)
    for n in (2, 1200):
        off, tok = batch_of(wf, n, [[0] * 100])
        log_z, status, tape = wf.forward(d, off, tok)
        assert bool((status == 0).all())
        with pytest.raises(wf.WfstError) as e:
            wf.backward(d, tape)
        assert e.value.code == wf.WFST_EUNSUPPORTED
        tape.free()
    assert d.health() == 0


def _near(got, want, n_k):
    """Both within 1e-4 (log Z, relative) and 1e-5 a visit (counts) of the exact values."""
    import torch
    torch.cuda.synchronize()
    lz, post, st = (x.cpu().numpy().astype(np.float64) for x in got)
    wlz, wpost, wst = (x.cpu().numpy().astype(np.float64) for x in want)
    assert np.array_equal(st, wst)
    ok = wst == 0
    assert np.all(np.abs(lz[ok] - wlz[ok]) <= 2e-4 * np.maximum(1, np.abs(wlz[ok])))
    assert np.all(np.abs(post - wpost) <= 2e-5 * np.maximum(1, n_k))


def _visits(fst, tok):
    return np.bincount(tok.cpu().numpy(), minlength=fst.num_ilabels)[fst.ilabel]


def test_no_room_for_lists(wf):
    """Without room for the lists of live states (here 74 kB; the streaming
    sweeps' largest buffer is 47 kB) the streaming sweeps run: the same paths,
    and log Z and counts as accurate; and the lists again once there is room."""
    say("case: no room for lists")
    fst = fan(23, 20, 30, seed=5)
    off, tok = batch_of(wf, 3)
    ref = wf.Fst.from_synth(fst)
    want_v, want = bits(wf.viterbi(ref, off, tok)), wf.forward_backward(ref, off, tok)
    d = wf.Fst.from_synth(fst)
    d.debug_alloc_limit(60000)
    assert bits(wf.viterbi(d, off, tok)) == want_v
    _near(wf.forward_backward(d, off, tok), want, _visits(fst, tok))
    d.debug_alloc_limit(0)
    assert bits(wf.viterbi(d, off, tok)) == want_v
    assert bits(wf.forward_backward(d, off, tok)) == bits(want)
    assert d.health() == 0


def test_no_room_for_narrow_tables_or_accumulators(wf):
    """The same for the forward pass over narrow labels (lookups of 8 bytes a
    token and destination, streaming tape 4), and for a backward pass without
    room for the accumulators (8 bytes an arc): the streaming sweeps run the
    forward pass again and take the counts."""
    say("case: no room for narrow tables, then for accumulators")
    fst, batch = synth.config(4, n_tags=45, vocab=400, batch=60, max_len=160)
    import torch
    off = torch.as_tensor(batch.offsets.astype(np.int32), device="cuda")
    tok = torch.as_tensor(batch.tokens, device="cuda")
    n, segs = tok.numel(), int(max(wf.Fst.from_synth(fst).label_stats()[1]))
    want = wf.forward_backward(wf.Fst.from_synth(fst), off, tok)
    d = wf.Fst.from_synth(fst)
    d.debug_alloc_limit(8 * n * segs - 1)
    lz, st, tape = wf.forward(d, off, tok)
    d.debug_alloc_limit(0)
    _near((lz, wf.backward(d, tape), st), want, _visits(fst, tok))
    tape.free()
    one_off, one_tok = off[:2].contiguous(), tok[:int(off[1])].contiguous()
    want = wf.forward_backward(wf.Fst.from_synth(fst), one_off, one_tok)
    d = wf.Fst.from_synth(fst)
    lz, st, tape = wf.forward(d, one_off, one_tok)
    d.debug_alloc_limit(8 * fst.num_arcs - 1)
    _near((lz, wf.backward(d, tape), st), want, _visits(fst, one_tok))
    tape.free()
    d.debug_alloc_limit(0)
    assert bits(wf.forward_backward(d, one_off, one_tok)) == bits(want)
    assert d.health() == 0


def test_no_room_for_lattice_lists(wf):
    """Kept lists of a lattice's nodes (12 bytes a state and node, against 4 of the whole vectors)."""
    say("case: no room for lattice lists")
    fst = fan(203, 200, 9, seed=6)
    nodes = 40
    arcs = [(v, v + 1, [1, 1, 2, 3][v % 4] if v else 0, -0.1 * k) for v in range(nodes - 1) for k in range(3)]
    flat = wf.lattices_from_lists([(nodes, arcs)] * 3)
    ref, st = (x.cpu().numpy() for x in wf.lattice_forward(wf.Fst.from_synth(fst), *flat))
    d = wf.Fst.from_synth(fst)
    d.debug_alloc_limit(4 * 3 * nodes * 204 + 1000)
    lz, st2 = (x.cpu().numpy() for x in wf.lattice_forward(d, *flat))
    assert np.array_equal(st, st2) and np.all(st == 0)
    assert np.all(np.abs(lz.astype(np.float64) - ref) <= 2e-4 * np.maximum(1, np.abs(ref)))
    d.debug_alloc_limit(0)
    assert (wf.lattice_forward(d, *flat)[0].cpu().numpy() == ref).all()
    assert d.health() == 0
