"""Passes over an FST whose state vectors exceed LDS, captured by the caller.

One eager call of the same shape sizes every buffer (as for FSTs that fit):
the capture allocates nothing, and replays, with eager work in between, give
the eager call's results, also for sentences that outgrow the lists.
"""
import gc

import numpy as np
import pytest

from gpu_common import say
from test_gpu_failed_calls import STRINGS, batch_of, bits, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import torch
    import paper_1701_03038_amd as wf
    assert torch.cuda.is_available()
    wf.load_library()
    return wf


@pytest.mark.parametrize("what", ["viterbi", "forward_backward"])
@pytest.mark.parametrize("n", [40, 900, 7000])
def test_capture_after_eager(wf, n, what):
    """n live states: lists of a wavefront, of a workgroup, and (7000 of 25011,
    more than a quarter) the streaming sweeps."""
    import torch
    say(f"case: wide capture {what} n={n}")
    fst = fan(25011, n, 90, seed=n)
    off, tok = batch_of(wf, 2)
    call = {"viterbi": lambda d: wf.viterbi(d, off, tok),
            "forward_backward": lambda d: wf.forward_backward(d, off, tok, final_posteriors=True)}[what]
    d = wf.Fst.from_synth(fst)
    want = [x.cpu().numpy() for x in call(d)]
    gc.collect()  # an earlier test's FST, freed in the middle of a capture, would synchronise the device and end it
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = call(d)
    for _ in range(3):
        for x in out:
            x.zero_()
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, want):
            x = x.cpu().numpy()
            if what == "viterbi" or x.dtype == np.int32:
                assert x.tobytes() == y.tobytes()
            else:  # the streaming forward pass runs as teams outside captures only: FP32 state on either side
                np.testing.assert_allclose(x, y, rtol=2e-4, atol=2e-5 * len(STRINGS) * 8)
        assert bits(call(d)) == [y.tobytes() for y in want]
    assert d.health() == 0
