"""A width's product and the sums that wait for it in one launch (csrc/gemm_step.hip), at the sizes where it can go wrong: spans that
fill, cross and miss a tile (15 or 31 sums), one to more than 32 terms, sentences that end inside a tile or have one span, bands before
and after, widths in this form next to widths in the others, one grammar per sentence, n_max past the longest sentence.
Against the CPU oracle with the tolerances of tests/parity_util.py."""
import numpy as np
import pytest

from oracle import spcfg_oracle as O
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth
from parity_util import check_all, check_grad, check_logZ

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,lens,more", [
    (1, 1, [2], 0),                     # the smallest call: no product of spans at all
    (30, 60, [16, 15, 17, 2, 3], 0),    # 15 and 16 starts: one tile, a tile and a span
    (30, 60, [31, 32, 1 + 31, 5], 3),   # two tiles and their remainders; roots are not the widest spans of the call
    (129, 500, [37, 21, 2], 0),         # more K-steps than wavefronts for the leaves, fewer for the spans
    (512, 512, [20], 0),                # the longest K, forward and reverse
    (64, 33, [33] * 40, 0),             # tall tiles, then small ones: 31 sums and 1, more than 256 small workgroups
    (100, 20, [34, 33, 2] * 12, 0),     # the same with two blocks of 64 nonterminals and mixed lengths
    (65, 30, [70], 0),                  # bands of four widths between, partial sums on both sides
    (20, 10, [45] * 50, 0),             # early widths apart, late ones together
])
def test_shared_grammar(N, P, lens, more):
    d = synth.make_inputs("tiny", seed=5400 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=90)
    if more:
        d["log_emit"] = np.concatenate([d["log_emit"], np.full((d["B"], more, P), np.nan, np.float32)], axis=1)
        d["n_max"] += more
    print("case step", N, P, lens[:4], len(lens), flush=True)
    wl = bd.Workload(d)
    wl.workspace.fill_(255)  # nothing is read before it is written
    g = np.linspace(-1.0, 2.0, len(lens)).astype(np.float32)  # (a zero and negative weights among them)
    for weights in (None, g):
        t = None if weights is None else wl.torch.from_numpy(weights).to(wl.logZ.device)
        wl.forward_backward(t)
        first = wl.results()
        check_all(first, O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"], grad_logZ=weights))
        wl.forward_backward(t)
        for k, v in wl.results().items():
            assert np.array_equal(v, first[k]), f"{k}: two runs differ bitwise"


def test_one_grammar_per_sentence():
    lens = [18, 2, 33, 16]
    d = synth.make_inputs_per_sentence("tiny", seed=5500, pad_value=np.nan, N=70, P=40, B=len(lens), lengths=lens)
    print("case step per sentence", flush=True)
    wl = bd.Workload(d)
    wl.forward_backward(None)
    got = wl.results()
    for b in range(len(lens)):
        n = int(d["lengths"][b])
        lz, gL, gR, gr, ge = O.inside_backward_sentence(d["log_root"][b], d["L"][b], d["R"][b], d["log_emit"][b, :n], 1.0)
        check_logZ(got["logZ"][b:b + 1], np.array([lz]))
        for name, x, y in (("grad_L", got["grad_L"][b], gL), ("grad_R", got["grad_R"][b], gR),
                           ("grad_log_root", got["grad_log_root"][b], gr), ("grad_log_emit", got["grad_log_emit"][b, :n], ge)):
            check_grad(name, x, y)
