"""The autotuner on batches that run over lists of live states.

Workgroup size, chunk length and the choice between records and fixed point
do not change their launches, so nothing may be picked among those by timing
noise; and a cache entry made for the streaming sweeps may not send them there.
"""
import json

import numpy as np
import pytest

import synth
from gpu_common import assert_fb_parity, assert_viterbi_parity, say
from test_gpu_failed_calls import batch_of, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


@pytest.mark.parametrize("case", ["narrow", "lists"])
def test_same_launches_share_one_timing(wf, case):
    say(f"case: autotune {case}")
    fst, batch = (synth.config(4, vocab=3000, batch=64, max_len=40) if case == "narrow" else
                  synth.config(2, vocab=200, batch=24))
    d = wf.Fst.from_synth(fst, chunk_arcs=16, threads_per_sentence=512)
    r = d.autotune(batch.offsets, batch.tokens, tune_chunk=case == "narrow")
    live = {v for (c, nt, path), v in r["times"].items() if path != "grouped"}
    assert len(live) == 1, r["times"]
    assert r["tried"] == len(r["times"])
    if r["count_path"] != "grouped":
        assert (r["chunk_arcs"], r["threads_per_sentence"], r["count_path"]) == (16, 512, "records")
    assert_viterbi_parity(fst, batch, d, ctx=case)
    assert_fb_parity(fst, batch, d, ctx=case)


def test_left_sentences_are_timed_one_by_one(wf):
    say("case: autotune with sentences left over")
    fst = fan(203, 200, 90, seed=3)
    d = wf.Fst.from_synth(fst)
    off, tok = batch_of(wf, 40)
    r = d.autotune(off, tok)
    assert len({v for (c, nt, path), v in r["times"].items() if path != "grouped"}) > 1, r["times"]


def test_cache_entries_of_streaming_sweeps_are_not_applied(wf, tmp_path):
    say("case: cache written without the index")
    fst, batch = synth.config(4, vocab=3000, batch=64, max_len=40)
    cache = str(tmp_path / "tune.json")
    wf.Fst.from_synth(fst).autotune(batch.offsets, batch.tokens, cache_path=cache)
    (key,) = json.load(open(cache))
    wf.Fst.from_synth(fst, state_memory=2).autotune(batch.offsets, batch.tokens, cache_path=cache)
    keys = list(json.load(open(cache)))
    assert len(keys) == 2 and key in keys
    (other,) = [k for k in keys if k != key]
    with open(cache, "w") as f:
        f.write('{\n"%s": {"threads_per_sentence": 64, "count_records": -1, "chunk_arcs": 16, "ms": 0.0010}\n}\n' % other)
    d = wf.Fst.from_synth(fst)
    r = d.autotune(batch.offsets, batch.tokens, cache_path=cache)
    assert not r["from_cache"]
    assert np.array_equal(wf.viterbi(d, batch.offsets, batch.tokens)[2].cpu().numpy() == 0, np.ones(batch.size, bool))
