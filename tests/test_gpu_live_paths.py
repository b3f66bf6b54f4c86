"""Forms of the passes over live states that need particular sizes.

State vectors beyond LDS with lists beyond a wavefront's (the workgroup forms,
and the streaming sweeps with team forward), after score updates; and sizes
whose forward vectors fit LDS while the backward sweep's do not, so that
sentences left over take the global-memory backward sweep over a device list.
"""
import gc

import numpy as np
import pytest

import oracle
import synth
from gpu_common import assert_fb_parity, assert_final_parity, assert_viterbi_parity, say
from test_gpu_failed_calls import STRINGS, batch_of, bits, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


@pytest.mark.parametrize("n,copies", [(40, 2), (900, 2), (900, 40), (7000, 2)])
def test_new_scores_of_wide_fsts(wf, n, copies):
    """After set_scores every pass gives the bits of an FST created with the
    new scores, whichever pass comes first: lists of a wavefront, of a
    workgroup (every sentence, or those a wavefront gave up), and 7000 of 25011
    states, where the sliced layouts' copies have to follow; eagerly and in a
    graph made before the update."""
    import torch
    say(f"case: new scores, wide n={n} copies={copies}")
    fst = fan(25011, n, 90, seed=n)
    off, tok = batch_of(wf, copies)
    passes = [lambda d: wf.viterbi(d, off, tok), lambda d: wf.forward_backward(d, off, tok, final_posteriors=True)]
    rng = np.random.default_rng(n)
    d = wf.Fst.from_synth(fst)
    graph = wf.Graph(d, off, tok)
    for step in range(2):
        new = (fst.arc_score + rng.normal(0, 0.3, fst.num_arcs)).astype(np.float32)
        new[rng.integers(0, new.size)] = -0.0
        f2 = synth.Fst(**{**fst.__dict__})
        f2.arc_score = new
        ref = wf.Fst.from_synth(f2)
        d.set_scores(torch.tensor(new, device="cuda"))
        for run in passes[step:] + passes[:step]:
            assert bits(run(d)) == bits(run(ref))
        d.set_scores(torch.tensor(fst.arc_score, device="cuda"))
        d.set_scores(torch.tensor(new, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        assert bits((graph.best_score, graph.best_arcs)) == bits(wf.viterbi(ref, off, tok)[:2])
        assert d.health() == 0
    graph.close()


@pytest.mark.parametrize("n,copies", [(40, 3), (90, 3), (90, 30), (500, 3)])
def test_left_sentences_with_backward_in_global_memory(wf, n, copies):
    """13000 states: forward vectors fit LDS, the backward sweep's do not.
    Lists up to 64 states stay, longer ones are left over; parity, weights of
    both signs, and the same bits from a graph, from fixed-point counts and on
    repeats."""
    import torch
    say(f"case: backward of left sentences in global memory n={n} copies={copies}")
    fst = fan(13000, n, 70, seed=n)
    off, tok = batch_of(wf, copies)
    batch = synth.Batch(off.cpu().numpy().astype(np.int64), tok.cpu().numpy())
    d = wf.Fst.from_synth(fst)
    assert_viterbi_parity(fst, batch, d, f"n={n}")
    assert_fb_parity(fst, batch, d, f"n={n}")
    assert_final_parity(fst, batch, d, f"n={n}")
    want = bits(wf.forward_backward(d, off, tok, final_posteriors=True))
    for other in (d, wf.Fst.from_synth(fst, count_records=-2), wf.Fst.from_synth(fst, checkpoint=1)):
        assert bits(wf.forward_backward(other, off, tok, final_posteriors=True)) == want
    g = wf.Graph(d, off, tok, final=True)
    for _ in range(3):
        g.replay()
        assert bits((g.log_z, g.grad, g.grad_final, g.status)) == want
        wf.viterbi(d, off, tok)
    g.close()
    lz, st, tape = wf.forward(d, off, tok)
    w = np.linspace(-1.0, 2.0, batch.size)
    w[st.cpu().numpy() != 0] = 0.0
    post, fin = wf.backward(d, tape, torch.tensor(w.astype(np.float32), device="cuda"), final=True)
    torch.cuda.synchronize()
    tape.free()
    _, opost, ofin, _ = oracle.forward_backward(fst, batch, grad_log_z=w.astype(np.float32).astype(np.float64),
                                                final_posteriors=True)
    n_k = np.bincount(batch.tokens, minlength=fst.num_ilabels)[fst.ilabel]
    assert np.all(np.abs(post.cpu().numpy() - opost) <= 2e-5 * np.maximum(1, n_k))
    assert np.all(np.abs(fin.cpu().numpy() - ofin) <= 2e-5 * batch.size)
    assert d.health() == 0


@pytest.mark.parametrize("n", [90, 500])
def test_capture_with_backward_in_global_memory(wf, n):
    """... and captured by the caller after one eager call."""
    import torch
    say(f"case: capture, backward in global memory n={n}")
    fst = fan(13000, n, 70, seed=n)
    off, tok = batch_of(wf, 2)
    d = wf.Fst.from_synth(fst)
    want = bits(wf.forward_backward(d, off, tok))
    gc.collect()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = wf.forward_backward(d, off, tok)
    for _ in range(3):
        for x in out:
            x.zero_()
        g.replay()
        assert bits(out) == want
        wf.viterbi(d, off, tok)
    assert len(STRINGS) * 2 == off.numel() - 1 and d.health() == 0
