"""The calls whose speed counts: the work a program has this library do.

Each case is a public call (or the few calls of one training step) on a
synthetic WFST of the families this repository builds and benchmarks: HMM
taggers written as WFSTs (bigram and trigram, 12 to 45 tags, vocabularies up to
200k), power-law WFSTs up to 1M states and 50M arcs, and confusion networks as
input lattices.  The WFST of a case is a function of its sizes alone (a program
loads its transducer once and decodes many batches with it); sentences,
lattices and training scores are drawn from the seed.

listed()  the cases; draw(rng) one more of the same ranges
prepare() what a program holds before the call; run() one pass; work() what a
pass can not do without; exact() the same outputs in 64 bits from plain torch.
"""
import math
from collections import OrderedDict

import numpy as np
import torch

DEV = "cuda"


def listed():
    tri = dict(fst="trigram", tags=45, vocab=50000)
    big = dict(fst="bigram", tags=45, vocab=200000)
    return [
        # one short sentence decoded at a time: an interactive tagger
        dict(name="decode_one_bigram12", call="decode", fst="bigram", tags=12, vocab=1000, batch=1, lo=30, hi=30),
        # posteriors of one sentence on the large tagger: active learning, per-sentence EM
        dict(name="posteriors_one_trigram", call="posteriors", batch=1, lo=25, hi=25, **tri),
        # the latency entry point for one long sentence on a small state space
        dict(name="scan_one_bigram", call="scan", batch=1, lo=200, hi=200, **big),
        # tagging a corpus, the repository's main batch (lognormal lengths, mean 25)
        dict(name="decode_batch_trigram", call="decode", batch=4096, lo=5, hi=60, **tri),
        # expected counts of the same batch, final-state posteriors among them
        dict(name="posteriors_batch_trigram", call="posteriors", batch=4096, lo=5, hi=60, **tri),
        # one training step: new scores, log Z of every sentence, gradient in every arc score
        dict(name="train_trigram", call="train", batch=1024, lo=5, hi=60, **tri),
        # rescoring recogniser output: log Z of the tagger composed with confusion networks
        dict(name="lattice_trigram", call="lattice", batch=4096, lo=5, hi=60, alternatives=3, **tri),
        # many ragged sentences on a small state space and a large vocabulary
        dict(name="decode_batch_bigram", call="decode", batch=16384, lo=1, hi=200, **big),
        dict(name="posteriors_batch_bigram", call="posteriors", batch=16384, lo=1, hi=200, **big),
        # one EM iteration: new scores, expected counts, normalisation per state
        dict(name="em_bigram", call="em", batch=4096, lo=1, hi=200, **big),
        # a transducer whose state vectors exceed on-chip memory: training step on random-walk strings
        dict(name="train_powerlaw", call="train", fst="powerlaw", states=1000000, arcs=50000000, labels=10000,
             batch=24, lo=100, hi=100),
        # few labels, so that every step can occupy most states (no sparsity to use)
        dict(name="posteriors_saturated", call="posteriors", fst="powerlaw", states=2000, arcs=100000, labels=20,
             batch=512, lo=5, hi=60),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["bigram", "bigram", "trigram", "trigram", "powerlaw"])
    if kind == "bigram":
        c = dict(call=rng.choice(["decode", "posteriors", "em", "scan", "train"]), fst="bigram", tags=rng.randint(12, 45),
                 vocab=_log_int(rng, 1000, 200000), batch=_log_int(rng, 1, 8192), lo=1, hi=rng.randint(20, 200))
        if c["call"] == "scan":
            c["batch"] = _log_int(rng, 1, 16)
    elif kind == "trigram":
        c = dict(call=rng.choice(["decode", "posteriors", "lattice", "train"]), fst="trigram", tags=rng.randint(12, 45),
                 vocab=_log_int(rng, 500, 20000), batch=_log_int(rng, 1, 4096), lo=rng.randint(1, 8),
                 hi=rng.randint(30, 60))
        if c["call"] == "lattice":
            c["alternatives"] = rng.randint(1, 4)
    else:
        states = _log_int(rng, 1000, 200000)
        c = dict(call=rng.choice(["decode", "posteriors", "train"]), fst="powerlaw", states=states,
                 arcs=states * rng.randint(30, 50), labels=_log_int(rng, 20, 10000) if states < 8000 else
                 _log_int(rng, 1000, 10000), batch=_log_int(rng, 1, 256) if states < 8000 else _log_int(rng, 1, 16),
                 lo=5, hi=rng.randint(30, 60))
    return c


# ------------------------------------------------------------------ inputs

class _Arcs:
    """A WFST as device arrays, arc id = index."""

    def __init__(self, Q, M, src, dst, lab, score, final):
        self.Q, self.M, self.start = Q, M, 0
        self.src, self.dst, self.lab, self.score, self.final = src, dst, lab, score, final
        self._index = None

    @property
    def A(self):
        return self.src.numel()

    def index(self):
        """Arc ids grouped by (label, source) and the keys label * Q + source, for exact()."""
        if self._index is None:
            key = self.lab.long() * self.Q + self.src
            if bool((key[1:] < key[:-1]).any()):
                key, order = torch.sort(key, stable=True)
            else:
                order = None
            self._index = (key, order)
        return self._index


def _gamma(rng, alpha, shape):
    g = rng.gamma(alpha, 1.0, shape)
    return np.maximum(g, np.finfo(np.float64).tiny)


def _tagger(order, tags, vocab):
    """HMM tagger: arc (context, word:tag) -> next context for every context and
    every tag of the word, score log p(tag | context) + log p(word | tag)."""
    rng = np.random.default_rng([order, tags, vocab])
    if order == 2:
        c, alpha = rng.integers(1, 4, vocab), 1.0
    else:
        c, alpha = np.minimum(rng.geometric(0.6, vocab), 8), 0.5
    c = np.minimum(c, tags)
    choice = np.argsort(rng.random((vocab, tags), dtype=np.float32), axis=1)[:, :8]
    word = np.repeat(np.arange(vocab), c)
    first = np.cumsum(c) - c
    tag = choice[word, np.arange(word.size) - np.repeat(first, c)]
    g = _gamma(rng, alpha, word.size)
    emit = np.log(g) - np.log(np.bincount(tag, weights=g, minlength=tags))[tag]
    Q = 1 + tags if order == 2 else 1 + tags + tags * tags
    g = _gamma(rng, alpha, (Q, tags))
    trans = np.log(g) - np.log(g.sum(1, keepdims=True))
    t = np.arange(tags)
    if order == 2:
        nxt = np.broadcast_to(1 + t, (Q, tags))
    else:
        last = np.concatenate([np.zeros(1, np.int64), t, np.tile(t, tags)])  # last tag of each context
        nxt = 1 + tags + tags * last[:, None] + t[None, :]
        nxt[0] = 1 + t
    up = lambda x: torch.as_tensor(np.ascontiguousarray(x), device=DEV)  # noqa: E731
    cd, fd, tagd, emitd, transd, nxtd = up(c), up(first), up(tag), up(emit), up(trans), up(nxt)
    size = cd * Q
    lab = torch.repeat_interleave(torch.arange(vocab, device=DEV), size)
    within = torch.arange(lab.numel(), device=DEV) - (torch.cumsum(size, 0) - size)[lab]
    src = within // cd[lab]
    pair = fd[lab] + within % cd[lab]
    del within
    dst = nxtd[src, tagd[pair]]
    score = (transd[src, tagd[pair]] + emitd[pair]).float()
    return _Arcs(Q, vocab, src.int(), dst.int(), lab.int(), score, torch.zeros(Q, device=DEV))


def _zipf_cdf(n, s):
    p = torch.arange(1, n + 1, device=DEV, dtype=torch.float64) ** -s
    return torch.cumsum(p, 0) / p.sum()


def _zipf(gen, cdf, shape):
    u = torch.rand(shape, generator=gen, device=DEV, dtype=torch.float64)
    return torch.searchsorted(cdf, u, right=True).clamp_(max=cdf.numel() - 1)


def _powerlaw(states, arcs, labels):
    """Out-degrees ~ d^-2.1 on [10, 5000] topped up to `arcs`, uniform
    destinations, Zipf(1) labels, scores -Exp(1), every state final."""
    gen = torch.Generator(DEV).manual_seed(states * 31 + labels)
    hi = min(5000, states)
    p = torch.arange(10, hi + 1, device=DEV, dtype=torch.float64) ** -2.1
    cdf = torch.cumsum(p, 0) / p.sum()
    deg = 10 + torch.searchsorted(cdf, torch.rand(states, generator=gen, device=DEV, dtype=torch.float64)).clamp_(max=hi - 10)
    while int(deg.sum()) > arcs:  # few arcs per state: a shorter tail, and still 10 arcs or more from every state
        hi //= 2
        deg.clamp_(max=hi)
    src = torch.repeat_interleave(torch.arange(states, device=DEV), deg)
    extra = arcs - src.numel()
    if extra > 0:
        more = torch.randint(0, states, (extra,), generator=gen, device=DEV)
        src = torch.sort(torch.cat([src, more]))[0]
    dst = torch.randint(0, states, (arcs,), generator=gen, device=DEV)
    lab = _zipf(gen, _zipf_cdf(labels, 1.0), (arcs,))
    score = torch.log(torch.rand(arcs, generator=gen, device=DEV).clamp_min_(1e-30))
    return _Arcs(states, labels, src.int(), dst.int(), lab.int(), score, torch.zeros(states, device=DEV))


_kept = OrderedDict()  # the last WFSTs by their sizes: [arcs, library handle or None]


def _wfst(case, handle):
    """The case's WFST and (with handle) its Fst: loaded once, as a program does."""
    key = tuple(case.get(k) for k in ("fst", "tags", "vocab", "states", "arcs", "labels"))
    if key not in _kept:
        while _kept:
            _, (_, old) = _kept.popitem()
            if old is not None:
                old.close()
        if case["fst"] == "powerlaw":
            a = _powerlaw(case["states"], case["arcs"], case["labels"])
        else:
            a = _tagger(2 if case["fst"] == "bigram" else 3, case["tags"], case["vocab"])
        _kept[key] = [a, None]
    got = _kept[key]
    if handle and got[1] is None:
        import paper_1701_03038_amd as wf
        a = got[0]
        host = [x.cpu().numpy() for x in (a.src, a.dst, a.lab, a.score, a.final)]
        torch.cuda.empty_cache()
        got[1] = wf.Fst(a.Q, a.M, a.start, *host[:3], host[3], host[4], olabel=host[2])
    return got


def _lengths(case, seed):
    """Sentence lengths: the case's own multiset (so that batches have equal sizes), in the seed's order."""
    lo, hi, n = case["lo"], case["hi"], case["batch"]
    rng = np.random.default_rng([lo, hi, n])
    if case["fst"] == "trigram" and n > 1:  # sentence lengths of the main batch
        mu = math.log(25.0) - 0.125
        lens = np.clip(np.rint(rng.lognormal(mu, 0.5, n)), lo, hi).astype(np.int64)
    else:
        lens = rng.integers(lo, hi + 1, n)
    return np.random.default_rng([seed, 1]).permutation(lens)


def _inputs(case, arcs, seed):
    """offsets int32 [B+1] and tokens int32 [N] on the device."""
    gen = torch.Generator(DEV).manual_seed(seed)
    lens = _lengths(case, seed)
    off = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    if case["fst"] == "powerlaw":  # strings read off random walks, so that every string has a path
        out = torch.searchsorted(arcs.src, torch.arange(arcs.Q + 1, device=DEV, dtype=torch.int32))
        B, T = lens.size, int(lens.max())
        state = torch.full((B,), arcs.start, device=DEV, dtype=torch.long)
        u = torch.rand((T, B), generator=gen, device=DEV, dtype=torch.float64)
        walk = torch.empty((B, T), device=DEV, dtype=torch.int32)
        for t in range(T):
            k = out[state] + (u[t] * (out[state + 1] - out[state])).long()
            walk[:, t] = arcs.lab[k]
            state = arcs.dst[k].long()
        keep = torch.arange(T, device=DEV)[None, :] < torch.as_tensor(lens, device=DEV)[:, None]
        tok = walk[keep]
    else:
        tok = _zipf(gen, _zipf_cdf(arcs.M, 1.1), (int(off[-1]),)).int()
    return torch.as_tensor(off, device=DEV).int(), tok.contiguous()


def _networks(case, arcs, seed):
    """Confusion networks around the sentences, flat as lattice_forward takes
    them: slot t joins node t to t+1 with the token, `alternatives` Zipf-drawn
    competitors and, with probability 0.1, an epsilon arc."""
    off, tok = _inputs(case, arcs, seed)
    gen = torch.Generator(DEV).manual_seed(seed + 1)
    N, K = tok.numel(), case["alternatives"] + 2
    lab = torch.empty((N, K), device=DEV, dtype=torch.int32)
    lab[:, 0] = tok
    lab[:, 1:K - 1] = _zipf(gen, _zipf_cdf(arcs.M, 1.1), (N, K - 2)).int()
    lab[:, K - 1] = -1
    use = torch.ones((N, K), device=DEV, dtype=torch.bool)
    use[:, K - 1] = torch.rand(N, generator=gen, device=DEV) < 0.1
    g = -torch.log(torch.rand((N, K), generator=gen, device=DEV).clamp_min_(1e-30)) * use
    weight = torch.log((g / g.sum(1, keepdim=True)).clamp_min_(1e-30))
    sent = torch.repeat_interleave(torch.arange(off.numel() - 1, device=DEV), (off[1:] - off[:-1]).long())
    pos = torch.arange(N, device=DEV) - off.long()[sent]
    frm = pos[:, None].expand(N, K)[use].int()
    slots = torch.cat([torch.zeros(1, device=DEV, dtype=torch.long), torch.cumsum(use.sum(1), 0)])
    node_off = off + torch.arange(off.numel(), device=DEV, dtype=torch.int32)
    return node_off, slots[off.long()].int(), frm, frm + 1, lab[use].contiguous(), weight[use].contiguous(), off


def _theta(arcs, seed):
    gen = torch.Generator(DEV).manual_seed(seed + 2)
    return arcs.score + 0.1 * torch.randn(arcs.A, generator=gen, device=DEV)


def _weights(case, seed):
    return torch.linspace(0.5, 1.5, case["batch"], device=DEV) + (seed % 7) * 0.1


def prepare(case, seed):
    arcs, fst = _wfst(case, True)
    state = dict(call=case["call"], fst=fst)
    if case["call"] == "lattice":
        state["net"] = _networks(case, arcs, seed)[:6]
    else:
        state["off"], state["tok"] = _inputs(case, arcs, seed)
    if case["call"] in ("train", "em"):
        state["theta"] = _theta(arcs, seed).requires_grad_(case["call"] == "train")
        state["weight"] = _weights(case, seed)
    else:
        fst.set_scores(arcs.score)  # a training case may have left other scores
    return state


# -------------------------------------------------------------------- calls

def run(s):
    import paper_1701_03038_amd as wf
    fst, call = s["fst"], s["call"]
    if call == "decode":
        return wf.viterbi(fst, s["off"], s["tok"], olabels=True)
    if call == "posteriors":
        return wf.forward_backward(fst, s["off"], s["tok"], final_posteriors=True)
    if call == "scan":
        return wf.forward_scan(fst, s["off"], s["tok"], alpha=True)
    if call == "lattice":
        return wf.lattice_forward(fst, *s["net"])
    if call == "em":  # E-step and M-step under new scores
        fst.set_scores(s["theta"])
        log_z, counts, status = wf.forward_backward(fst, s["off"], s["tok"])
        return log_z, counts, status, wf.em_update(fst, counts, s["theta"], 0.1)
    theta = s["theta"]  # train
    theta.grad = None
    log_z, status = wf.log_partition(theta, fst, s["off"], s["tok"])
    (log_z * s["weight"]).sum().backward()
    return log_z.detach(), status, theta.grad


def work(case):
    """Tokens, live arcs ({state, score}, 8 bytes each) and outputs, each once.
    Live arcs per token of a tagger: one per tag of the word and of the words
    that make up the context."""
    B = case["batch"]
    mean = 25.0 if case["fst"] == "trigram" and B > 1 else (case["lo"] + case["hi"]) / 2
    N = B * mean
    c = 2.0 if case["fst"] == "bigram" else 1.66
    if case["fst"] == "powerlaw":
        A, Q = case["arcs"], case["states"]
        live = min(6.0 * N, A)
    else:
        order = 2 if case["fst"] == "bigram" else 3
        Q = 1 + case["tags"] + (case["tags"] ** 2 if order == 3 else 0)
        A = case["vocab"] * c * Q
        live = N * c ** order
    if case["call"] == "lattice":
        n = N * (case["alternatives"] + 1)
        return dict(bytes=16.0 * n + 8.0 * live * (case["alternatives"] + 1) ** 3 + 8.0 * B, flops=6.0 * n * c ** 3)
    out = dict(decode=8.0 * N + 8 * B, posteriors=4.0 * A + 4 * Q + 8 * B, scan=4.0 * N * Q + 8 * B,
               train=8.0 * A + 8 * B, em=12.0 * A + 8 * B)[case["call"]]
    return dict(bytes=4.0 * N + 8.0 * live + out, flops=(2.0 if case["call"] == "decode" else 12.0) * live)


# ------------------------------------------------------------ 64-bit results

def _expand(arcs, sent, state, label):
    """Every arc of `label[i]` leaving `state[i]`: (row i, arc id)."""
    key, order = arcs.index()
    k = label.long() * arcs.Q + state
    lo, hi = torch.searchsorted(key, k), torch.searchsorted(key, k, right=True)
    n = hi - lo
    row = torch.repeat_interleave(torch.arange(k.numel(), device=DEV), n)
    at = lo[row] + torch.arange(row.numel(), device=DEV) - (torch.cumsum(n, 0) - n)[row]
    return row, at if order is None else order[at]


def _reduce(key, x, best):
    """Values x grouped by key: (keys, max or log-sum-exp of each group, group of each value)."""
    u, inv = torch.unique(key, return_inverse=True)
    m = torch.full((u.numel(),), -math.inf, device=DEV, dtype=torch.float64).scatter_reduce_(0, inv, x, "amax")
    if best:
        return u, m, inv
    s = torch.zeros_like(m).index_add_(0, inv, torch.exp(x - m[inv]))
    return u, m + torch.log(s), inv


def _forward(arcs, score, off, tok, best=False):
    """Live (sentence, state) pairs and their value after each step, and the arcs between them."""
    off = off.long()
    T = off[1:] - off[:-1]
    live = torch.arange(T.numel(), device=DEV) * arcs.Q + arcs.start
    val = torch.zeros(T.numel(), device=DEV, dtype=torch.float64)
    end = [(live[T == 0], val[T == 0])]
    steps = []
    for t in range(int(T.max()) if T.numel() else 0):
        on = T[live // arcs.Q] > t
        live, val = live[on], val[on]
        sent, state = live // arcs.Q, live % arcs.Q
        i = off[sent] + t
        row, arc = _expand(arcs, sent, state, tok[i])
        x = val[row] + score[arc].double()
        nxt, v, inv = _reduce(sent[row] * arcs.Q + arcs.dst[arc].long(), x, best)
        steps.append((live, val, row, arc, inv, i[row]))
        live, val = nxt, v
        last = T[live // arcs.Q] == t + 1
        end.append((live[last], val[last]))
        steps[-1] += (live, val)
    live = torch.cat([e[0] for e in end])
    val = torch.cat([e[1] for e in end])
    fin = val + arcs.final.double()[live % arcs.Q]
    z = torch.full((T.numel(),), -math.inf, device=DEV, dtype=torch.float64)
    u, v, _ = _reduce(live // arcs.Q, fin, best)
    z[u] = v
    return z, steps, live, fin


def _counts(arcs, score, off, tok, weight):
    """(log Z, weighted expected counts of every arc, and of every final state)."""
    z, steps, live, fin = _forward(arcs, score, off, tok)
    T = (off[1:] - off[:-1]).long()
    Q = arcs.Q
    grad = torch.zeros(arcs.A, device=DEV, dtype=torch.float64)
    sent = live // Q
    gfin = torch.zeros(Q, device=DEV, dtype=torch.float64)
    gfin.index_add_(0, live % Q, weight[sent] * torch.exp(fin - z[sent]))
    beta = None
    for t in range(len(steps) - 1, -1, -1):
        here, val, row, arc, inv, _, nxt, _ = steps[t]
        b = torch.full((nxt.numel(),), -math.inf, device=DEV, dtype=torch.float64)
        ends = T[nxt // Q] == t + 1
        b[ends] = arcs.final.double()[nxt[ends] % Q]
        if beta is not None:
            b[~ends] = beta
        x = score[arc].double() + b[inv]
        sent = here[row] // Q
        grad.index_add_(0, arc, weight[sent] * torch.exp(val[row] + x - z[sent]))
        m = torch.full((here.numel(),), -math.inf, device=DEV, dtype=torch.float64).scatter_reduce_(0, row, x, "amax")
        s = torch.zeros_like(m).index_add_(0, row, torch.exp(x - m.clamp_min(-1e300)[row]))
        beta = m + torch.log(s)
    return z, grad, gfin


def _lattice(arcs, net):
    """log Z per confusion network: every slot of a network merges its arcs into one vector."""
    _, arc_off, frm, _, lab, weight, off = net
    B, Q = off.numel() - 1, arcs.Q
    T = (off[1:] - off[:-1]).long()
    sent = torch.repeat_interleave(torch.arange(B, device=DEV), (arc_off[1:] - arc_off[:-1]).long())
    slot, order = torch.sort(sent * 4096 + frm.long())
    live = torch.arange(B, device=DEV) * Q + arcs.start
    val = torch.zeros(B, device=DEV, dtype=torch.float64)
    z = torch.full((B,), -math.inf, device=DEV, dtype=torch.float64)
    for t in range(int(T.max())):
        s = live // Q
        k = s * 4096 + t
        lo, hi = torch.searchsorted(slot, k), torch.searchsorted(slot, k, right=True)
        n = hi - lo
        row = torch.repeat_interleave(torch.arange(k.numel(), device=DEV), n)
        e = order[lo[row] + torch.arange(row.numel(), device=DEV) - (torch.cumsum(n, 0) - n)[row]]
        x = val[row] + weight[e].double()
        eps = lab[e] < 0
        keys, vals = [live[row[eps]]], [x[eps]]
        row, e, x = row[~eps], e[~eps], x[~eps]
        r2, arc = _expand(arcs, s[row], live[row] % Q, lab[e])
        keys.append(s[row][r2] * Q + arcs.dst[arc].long())
        vals.append(x[r2] + arcs.score[arc].double())
        live, val, _ = _reduce(torch.cat(keys), torch.cat(vals), False)
        last = T[live // Q] == t + 1
        u, v, _ = _reduce(live[last] // Q, val[last] + arcs.final.double()[live[last] % Q], False)
        z[u] = v
        live, val = live[~last], val[~last]
    return z


def exact(case, seed):
    arcs = _wfst(case, False)[0]
    call = case["call"]
    if call == "lattice":
        return _lattice(arcs, _networks(case, arcs, seed)), None
    off, tok = _inputs(case, arcs, seed)
    if call == "decode":
        return _forward(arcs, arcs.score, off, tok, best=True)[0], None, None, None
    if call == "scan":
        z, steps, _, _ = _forward(arcs, arcs.score, off, tok)
        alpha = torch.full((tok.numel(), arcs.Q), -math.inf, device=DEV, dtype=torch.float64)
        for t, step in enumerate(steps):
            nxt, v = step[-2:]
            alpha[off.long()[nxt // arcs.Q] + t, nxt % arcs.Q] = v
        return z, None, alpha
    if call == "posteriors":
        z, grad, gfin = _counts(arcs, arcs.score, off, tok, torch.ones(case["batch"], device=DEV, dtype=torch.float64))
        return z, grad, gfin, None
    theta = _theta(arcs, seed)
    if call == "train":
        z, grad, _ = _counts(arcs, theta, off, tok, _weights(case, seed).double())
        return z, None, grad
    z, grad, _ = _counts(arcs, theta, off, tok, torch.ones(case["batch"], device=DEV, dtype=torch.float64))
    total = torch.zeros(arcs.Q, device=DEV, dtype=torch.float64).index_add_(0, arcs.src.long(), grad + 0.1)
    return z, grad, None, torch.log(grad + 0.1) - torch.log(total)[arcs.src.long()]
