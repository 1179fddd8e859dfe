"""The work that users have this library do, as cases that can be timed: scoring, training, parsing and the
rule-probability front-end, over the range of grammar sizes, batch sizes, sentence lengths, precisions and options
that the configurations, the tests and the benchmark of this repository use.

A case is a plain dict:
  kind          "eval"   spcfg_inside: log Z per sentence (perplexity of held-out text, reranking)
                "train"  spcfg_inside_forward_backward: log Z and every gradient (one training step)
                "parse"  the same, then span posteriors, labels and the best bracketing per sentence
                "rules"  spcfg_rules_forward and spcfg_rules_backward: scores -> rule probabilities, and back
  B, N, P, V    sentences, nonterminals, preterminals, vocabulary
  law, lo, hi   sentence lengths: "const" (hi), "uniform" on [lo, hi], "normal" (mean 22, sd 10, clamped to [lo, hi])
  scale         standard deviation of the scores whose row softmaxes are L and R
  precision     "fp32" or "bf16"
  per_sentence  one grammar per sentence (compound variant)
  single        bf16: single bf16 operands in the forward products too (SPCFG_FLAG_BF16_SINGLE_FORWARD)
"""
from __future__ import annotations

import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2310_14997_amd import binding as bd

_BASE = dict(kind="train", B=1, N=1, P=1, V=10000, law="uniform", lo=2, hi=2, scale=1.0, precision="fp32",
             per_sentence=False, single=False)


def _case(**kw):
    return {**_BASE, **kw}


def listed():
    return [
        # scoring a handful of short sentences with a small grammar: launches and latency are everything
        _case(name="tiny_eval", kind="eval", B=4, N=30, P=60, V=200, law="const", lo=10, hi=10),
        # training a small grammar whose sizes are multiples of nothing, on a small ragged batch
        _case(name="ragged_train", B=7, N=141, P=333, V=1999, lo=2, hi=37, scale=2.0),
        # training the usual small grammar: every launch is short
        _case(name="small_train", B=32, N=512, P=512, lo=10, hi=30),
        # the same with one grammar per sentence (compound variant): every sentence brings its own L and R
        _case(name="small_compound_train", B=32, N=512, P=512, lo=10, hi=30, per_sentence=True),
        # parsing treebank-like sentences with a mid-sized grammar: posteriors, labels and trees
        _case(name="mid_parse", kind="parse", B=64, N=1024, P=1024, law="normal", lo=2, hi=40, scale=2.0),
        # a single long sentence scored with a large grammar, as in interactive use
        _case(name="single_eval", kind="eval", B=1, N=2048, P=2048, law="const", lo=40, hi=40, scale=2.0),
        # the headline: one training step on a treebank-shaped batch with 2048 nonterminals
        _case(name="ptb_train", B=64, N=2048, P=2048, law="normal", lo=2, hi=40, scale=2.0),
        # likelihood of held-out text with the same grammar
        _case(name="ptb_eval", kind="eval", B=64, N=2048, P=2048, law="normal", lo=2, hi=40, scale=2.0),
        # paragraphs instead of sentences: the cubic split-point reduction dominates
        _case(name="long_train", B=4, N=1024, P=1024, lo=100, hi=200),
        # a large grammar at full length on bf16 operands
        _case(name="scaled_train", B=32, N=4096, P=4096, law="const", lo=40, hi=40, precision="bf16"),
        # the same in evaluation, where single bf16 operands are accurate enough
        _case(name="scaled_eval", kind="eval", B=32, N=4096, P=4096, law="const", lo=40, hi=40, precision="bf16",
              single=True),
        # what turns the networks' scores into the headline's inputs, and its gradients back into score gradients
        _case(name="ptb_rules", kind="rules", B=64, N=2048, P=2048, law="normal", lo=2, hi=40, scale=2.0),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    """One more case: any size between the smallest and the largest listed ones, at no more than the largest's cost."""
    limit = [max(x) for x in zip(*(_cost(c) for c in listed()))]
    while True:
        u, v = rng.random(), rng.random()
        c = _case(kind="train" if u < 0.45 else "eval" if u < 0.65 else "parse" if u < 0.8 else "rules")
        c["B"] = _log_int(rng, 1, 64)
        c["N"], c["P"] = _log_int(rng, 30, 4096), _log_int(rng, 60, 4096)
        c["V"] = _log_int(rng, 200, 10000)
        c["hi"] = _log_int(rng, 8, 200)
        c["law"] = rng.choice(["uniform", "const", "normal"] if 25 <= c["hi"] <= 60 else ["uniform", "const"])
        c["lo"] = c["hi"] if c["law"] == "const" else 2 if c["law"] == "normal" else rng.randint(2, c["hi"])
        c["scale"] = rng.choice([1.0, 2.0])
        if c["kind"] != "rules":
            # (trees are decoded from fp32 posteriors: bf16 ones flip nearly tied brackets)
            c["precision"] = "bf16" if v < 0.25 and c["kind"] != "parse" else "fp32"
            c["single"] = c["precision"] == "bf16" and c["kind"] == "eval" and rng.random() < 0.5
            c["per_sentence"] = rng.random() < 0.15
        if c["per_sentence"] and c["B"] * c["N"] * (c["N"] + c["P"]) > 3e8:
            continue
        if all(x <= most for x, most in zip(_cost(c), limit)):
            return c


def _cost(case):
    # matrix work (an fp32 product costs about 3.6 bf16 ones), boundary bytes, split-point sums
    w = work(case)
    return (w["flops"] * (1.0 if case["precision"] == "bf16" else 3.6), w["bytes"],
            case["N"] * _counts(_lengths(case))[2])


def _lengths(case):
    """Sentence lengths of a case: the quantiles of its law (so that every seed has the same work), unordered."""
    B, lo, hi = case["B"], case["lo"], case["hi"]
    q = (np.arange(B) + 0.5) / B
    if case["law"] == "const":
        n = np.full(B, hi)
    elif case["law"] == "uniform":
        n = lo + np.floor(q * (hi - lo + 1))
    else:
        n = np.clip(np.rint([NormalDist(22.0, 10.0).inv_cdf(float(x)) for x in q]), lo, hi)
    n = n.astype(np.int32)
    n[0] = n.max()  # small batches: the longest sentence is there whatever the quantiles are
    return np.random.default_rng(B * 1000 + hi).permutation(n)


def _counts(n):
    n = n.astype(np.int64)
    spans = int((n * (n - 1) // 2 - 1).sum())  # projected spans of width >= 2 (the root is not projected)
    terms = int(((n - 1) * n * (n + 1) // 6).sum())  # (span, split point) pairs
    return int(n.sum()), spans, terms


def work(case):
    N, P, V, B = case["N"], case["P"], case["V"], case["B"]
    M = N + P
    n = _lengths(case)
    words, spans, terms = _counts(n)
    if case["kind"] == "rules":
        # forward: L / R scores in, probabilities out, the emission table in, one vector per token out; backward:
        # probabilities and their gradients in, score gradients out, the emission table in, its gradient out
        nbytes = 4 * (2 * N * M * (2 + 3) + P * V * (1 + 2) + words * P * 2)
        flops = 2 * N * M * (4 + 4) + P * V * (2 + 4)
        return dict(bytes=nbytes, flops=flops)
    G = B if case["per_sentence"] else 1
    passes = 1 if case["kind"] == "eval" else 3
    # [L;R] products (forward; reverse and rule gradients cost as much each), split-point sums (2 flop a term and
    # nonterminal forward, 4 backward)
    flops = passes * (4 * N * N * spans + 4 * N * P * words + 2 * N * terms)
    nbytes = 4 * (2 * G * N * M + words * P)  # grammar and emissions in
    if passes == 3:
        nbytes *= 2  # their gradients out
    if case["kind"] == "parse":
        nbytes += 8 * B * int(n.max()) ** 2
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    # About four times the largest distance seen, over the listed cases and forty drawn ones, between two correct
    # evaluations: fp32: the default products against fp32 matrix instructions (another rounding of every product,
    # other summation orders; 2.0e-6, single values 1.6e-5, log Z alone 1.1e-7); bf16: against the fp32 path on the
    # same inputs (2.0e-3 and 7.1e-3, log Z alone 5.0e-6 and 5.3e-6); front-end: against 64-bit softmaxes and their
    # derivatives (2.2e-7; 2.8e-5 where p * (g - sum p g) cancels).  Labels and trees were always the same in fp32; a
    # label in a thousand is left to ties.
    if case["kind"] == "rules":
        return {"rel": 9e-7, "max": 1.1e-4}
    if case["kind"] == "eval":
        return {"rel": 2e-5, "max": 2.1e-5} if case["precision"] == "bf16" else {"rel": 4.4e-7, "max": 4.4e-7}
    if case["precision"] == "bf16":
        return {"rel": 8e-3, "max": 2.8e-2}
    return {"rel": 8e-6, "max": 6.4e-5, "differ": 0.001}


def _softmax_rows(z):
    return torch.softmax(z, dim=-1).contiguous()


def prepare(case, seed):
    """Inputs on the GPU, made from the seed alone, and the buffers that a user's program keeps between calls."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    N, P, V, B = case["N"], case["P"], case["V"], case["B"]
    M, lengths = N + P, _lengths(case)
    n_max = int(lengths.max())
    f = dict(dtype=torch.float32, device=dev)
    randn = lambda *shape: torch.randn(*shape, generator=gen, **f)
    real = (torch.arange(n_max)[None, :] < torch.from_numpy(lengths).long()[:, None]).to(dev)  # [B, n_max]
    # bounded Zipf(1.1) tokens
    p = torch.arange(1, V + 1, dtype=torch.float64) ** -1.1
    cdf = torch.cumsum(p / p.sum(), 0).to(dev)
    u = torch.rand(B, n_max, generator=gen, dtype=torch.float64, device=dev)
    tokens = torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1)

    if case["kind"] == "rules":
        st = dict(kind="rules", lengths=lengths, tokens=torch.where(real, tokens, -1).to(torch.int32).contiguous(),
                  root_logits=randn(N), L_logits=case["scale"] * randn(N, M), R_logits=case["scale"] * randn(N, M),
                  emis_logits=randn(P, V))
        # gradients of log Z as the inside pass returns them: non-negative, preterminal posteriors sum to one a token
        root = _softmax_rows(randn(N)) * B
        st["grads"] = [root, torch.rand(N, M, generator=gen, **f), torch.rand(N, M, generator=gen, **f),
                       _softmax_rows(2.0 * randn(B, n_max, P)) * real[:, :, None]]
        st["fwd"] = [torch.empty(N, **f), torch.empty(N, M, **f), torch.empty(N, M, **f),
                     torch.empty(B, n_max, P, **f), torch.empty(P, **f)]
        st["bwd"] = [torch.empty(N, **f), torch.empty(N, M, **f), torch.empty(N, M, **f), torch.empty(P, V, **f)]
        st["scratch"] = torch.empty(32, P, **f)
        return st

    sc = case["scale"]
    root, L, R = randn(N), sc * randn(N, M), sc * randn(N, M)
    if case["per_sentence"]:  # related grammars: shared scores plus half as much of each sentence's own
        root = root + 0.5 * randn(B, N)
        L = L + 0.5 * sc * randn(B, N, M)
        R = R + 0.5 * sc * randn(B, N, M)
    table = torch.log_softmax(randn(P, V), dim=-1)
    log_emit = table.t().contiguous()[tokens]  # [B, n_max, P]
    if case["per_sentence"]:
        log_emit = torch.log_softmax(log_emit + 0.5 * randn(B, n_max, P), dim=-1)
    log_emit = (log_emit * real[:, :, None]).contiguous()
    L, R = _softmax_rows(L), _softmax_rows(R)
    log_root = torch.log_softmax(root, dim=-1).contiguous()

    flags = bd.FLAG_PER_SENTENCE_GRAMMAR if case["per_sentence"] else 0
    flags |= bd.FLAG_BF16_SINGLE_FORWARD if case["single"] else 0
    precision = bd.PRECISION_BF16 if case["precision"] == "bf16" else bd.PRECISION_FP32
    cfg = bd.make_config(N, P, B, n_max, precision, flags)
    st = dict(kind=case["kind"], cfg=cfg, lengths=lengths, n_max=n_max, inputs=[log_root, L, R, log_emit],
              logZ=torch.empty(B, **f),
              workspace=torch.empty(bd.spcfg_workspace_bytes_for(cfg, lengths, n_max), dtype=torch.uint8, device=dev))
    if case["kind"] != "eval":
        st["grads"] = [torch.empty_like(L), torch.empty_like(R), torch.empty_like(log_root), torch.empty_like(log_emit)]
    if case["kind"] == "parse":
        st["span_post"] = torch.empty(B, n_max, n_max, **f)
        st["span_label"] = torch.empty(B, n_max, n_max, dtype=torch.int32, device=dev)
        st["spans"] = torch.empty(B, n_max - 1, 2, dtype=torch.int32, device=dev)
        st["score"] = torch.empty(B, **f)
        st["scratch"] = torch.empty(bd.spcfg_mbr_decode_scratch_bytes(B, n_max), dtype=torch.uint8, device=dev)
    return st


def run(state):
    s = state
    if s["kind"] == "rules":
        log_root, L, R, log_emit, lse = s["fwd"]
        bd.spcfg_rules_forward(s["root_logits"], s["L_logits"], s["R_logits"], s["emis_logits"], s["tokens"],
                               s["lengths"], log_root, L, R, log_emit, lse)
        bd.spcfg_rules_backward(log_root, L, R, s["emis_logits"], lse, s["tokens"], s["lengths"], *s["grads"],
                                *s["bwd"], s["scratch"])
        return dict(log_root=log_root, L=L, R=R, log_emit=log_emit, grad_root=s["bwd"][0], grad_L=s["bwd"][1],
                    grad_R=s["bwd"][2], grad_emis=s["bwd"][3])
    if s["kind"] == "eval":
        bd.spcfg_inside(s["cfg"], *s["inputs"], s["lengths"], s["logZ"], s["workspace"])
        return s["logZ"]
    grad_L, grad_R, grad_log_root, grad_log_emit = s["grads"]
    bd.spcfg_inside_forward_backward(s["cfg"], *s["inputs"], s["lengths"], None, s["logZ"], grad_L, grad_R,
                                     grad_log_root, grad_log_emit, s["workspace"])
    out = dict(logZ=s["logZ"], grad_L=grad_L, grad_R=grad_R, grad_log_root=grad_log_root, grad_log_emit=grad_log_emit)
    if s["kind"] == "parse":
        bd.spcfg_span_marginals(s["cfg"], s["lengths"], s["n_max"], s["workspace"], s["span_post"], s["span_label"])
        bd.spcfg_mbr_decode(s["span_post"], s["lengths"], s["spans"], s["score"], s["scratch"])
        out.update(span_post=s["span_post"], span_label=s["span_label"], spans=s["spans"], score=s["score"])
    return out


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits: plain torch over dense slices, one per span width.

    Everything is in probability space.  Emissions are taken relative to their mean over the preterminals, token by
    token, and a span's weight then falls off like a power of its width, which 64 bits hold without scaling.  Labels
    and trees are whole numbers that ties may change: None.
    """
    if case["kind"] == "rules":
        return _exact_rules(case, seed)
    st = prepare(case, seed)
    N, P, n_max = case["N"], case["P"], st["n_max"]
    if case["B"] * n_max * n_max * (N + P) * 24 > 1e11:  # bytes of a chart and its adjoints: seconds of work, and room
        return None
    log_root, L, R, log_emit = [x.double() for x in st["inputs"]]
    real = (torch.arange(n_max)[None, :] < torch.from_numpy(st["lengths"]).long()[:, None]).to(log_emit.device)
    shift = torch.logsumexp(log_emit, -1) - math.log(P)  # [B, n_max]
    leaf = torch.exp(log_emit - shift[:, :, None]) * real[:, :, None]
    last = [(int(n), b) for b, n in enumerate(st["lengths"])]
    # project a [B, spans, .] slice through the columns of a factor that its kind of child has
    cols = lambda w: slice(N, N + P) if w == 1 else slice(0, N)
    proj = lambda beta, X, w: torch.matmul(beta, X[..., cols(w)].transpose(-1, -2).contiguous())

    beta, eta, zeta = {1: leaf}, {}, {}
    for w in range(1, n_max + 1):
        m = n_max - w + 1  # starts 0 .. m - 1
        if w >= 2:
            acc = torch.zeros(case["B"], m, N, dtype=torch.float64, device=leaf.device)
            for k in range(1, w):
                acc.addcmul_(eta[k][:, :m], zeta[w - k][:, k:k + m])
            beta[w] = acc
        if w < n_max:
            eta[w], zeta[w] = proj(beta[w], L, w), proj(beta[w], R, w)
    root = torch.exp(log_root)
    root = root if case["per_sentence"] else root.expand(case["B"], N)
    top = torch.stack([beta[n][b, 0] for n, b in last])
    Z = (root * top).sum(-1)
    logZ = torch.log(Z) + (shift * real).sum(-1)
    if case["kind"] == "eval":
        return logZ

    grad_log_root = root * top / Z[:, None]
    g_L, g_R = torch.zeros_like(L), torch.zeros_like(R)
    zeros = lambda w: torch.zeros(case["B"], n_max - w + 1, N, dtype=torch.float64, device=leaf.device)
    d_eta, d_zeta = {w: zeros(w) for w in eta}, {w: zeros(w) for w in zeta}
    post = torch.zeros(case["B"], n_max, n_max, dtype=torch.float64, device=leaf.device)
    for w in range(n_max, 0, -1):
        m = n_max - w + 1
        if w < n_max:
            for d, g, X in ((d_eta[w], g_L, L), (d_zeta[w], g_R, R)):
                if case["per_sentence"]:
                    g[..., cols(w)] += torch.matmul(d.transpose(-1, -2).contiguous(), beta[w])
                else:
                    g[..., cols(w)] += d.reshape(-1, N).t() @ beta[w].reshape(-1, beta[w].shape[-1])
            d_beta = torch.matmul(d_eta[w], L[..., cols(w)]) + torch.matmul(d_zeta[w], R[..., cols(w)])
        else:
            d_beta = zeros(w)
        if w >= 2:
            for n, b in last:
                if n == w:
                    d_beta[b, 0] += root[b] / Z[b]
            post[:, torch.arange(m), torch.arange(w - 1, n_max)] = (beta[w] * d_beta).sum(-1)
            for k in range(1, w):
                d_eta[k][:, :m].addcmul_(d_beta, zeta[w - k][:, k:k + m])
                d_zeta[w - k][:, k:k + m].addcmul_(d_beta, eta[k][:, :m])
            del beta[w], d_beta
    grad_log_emit = leaf * d_beta
    out = dict(logZ=logZ, grad_L=g_L, grad_R=g_R,
               grad_log_root=grad_log_root if case["per_sentence"] else grad_log_root.sum(0), grad_log_emit=grad_log_emit)
    if case["kind"] == "parse":
        best = {1: torch.zeros(case["B"], n_max, dtype=torch.float64, device=leaf.device)}
        for w in range(2, n_max + 1):
            m = n_max - w + 1
            kids = torch.stack([best[k][:, :m] + best[w - k][:, k:k + m] for k in range(1, w)])
            best[w] = post[:, torch.arange(m), torch.arange(w - 1, n_max)] + kids.amax(0)
        score = torch.stack([best[n][b, 0] for n, b in last])
        starts = torch.arange(n_max)
        post[:, starts, starts] = real.double()  # words are in every tree
        out.update(span_post=post, span_label=None, spans=None, score=score)
    return out


def _exact_rules(case, seed):
    st = prepare(case, seed)
    P, V = case["P"], case["V"]
    real = st["tokens"] >= 0
    tokens = st["tokens"].clamp_min(0).long()
    root, L, R, emis = [st[k].double() for k in ("root_logits", "L_logits", "R_logits", "emis_logits")]
    g_root, g_L, g_R, g_emit = [g.double() for g in st["grads"]]
    log_root, L, R, table = torch.log_softmax(root, -1), torch.softmax(L, -1), torch.softmax(R, -1), torch.log_softmax(emis, -1)
    back = lambda p, g: p * (g - (p * g).sum(-1, keepdim=True))
    # token by token into the table's gradient (positions past a sentence's end carry nothing)
    per_word = g_emit[real]  # [words, P]
    d_table = torch.zeros(V, P, dtype=torch.float64, device=emis.device).index_add_(0, tokens[real], per_word).t()
    return dict(log_root=log_root, L=L, R=R, log_emit=table.t()[tokens] * real[:, :, None],
                grad_root=g_root - torch.exp(log_root) * g_root.sum(), grad_L=back(L, g_L), grad_R=back(R, g_R),
                grad_emis=d_table - torch.exp(table) * per_word.sum(0)[:, None])
