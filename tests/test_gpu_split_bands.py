"""Bands of widths (k_split_band_fwd / k_split_band_bwd in csrc/kernels_elem.hip): partial split-point sums of four
widths in one pass, the rest by the launch of each width.  Against the CPU oracle, with the tolerances of
tests/parity_util.py, at the sizes where the bands' tables, tiles and ranges end; every case asserts which forms it reaches."""
import numpy as np
import pytest
import torch

import band_rule
from oracle import spcfg_oracle as O
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth
from parity_util import check_all, check_grad, check_logZ, oracle_batch_parallel

pytestmark = pytest.mark.gpu


# forms: wavefronts that share 64 nonterminals in the case's forward and reverse bands.  Sentences of 48 words and more take
# their late widths in bands whatever the grammar's size.
@pytest.mark.parametrize("N,P,lens,n_max,forms", [
    (7, 9, [49, 48, 2], None, ({16}, {16})),                # one band forward: its first width only, and only in one sentence
    (7, 9, [52, 51, 50, 53], 60, ({16}, {16})),             # band ends inside the longest sentence; padding beyond it
    (65, 20, [63, 17, 64, 3, 62], None, ({16}, {16})),      # two blocks of nonterminals; sentences shorter than every band
    (33, 10, [72, 68, 5], None, ({16}, {16})),              # the longest sentence's last width is in no band (k_split_fwd<4>)
    (200, 33, [57], 58, ({16}, {16})),                      # one sentence; n_max one above it
    (300, 65, [14] * 24 + [40] * 20, None, (set(), set())),  # too few rows saved for any band
    (310, 20, [48] * 60 + [21, 5], None, ({1}, {1})),       # five blocks of nonterminals dealt to six wavefronts; short sentences
    (180, 12, [60] * 70, None, ({1, 16}, {1})),             # three wavefronts a workgroup; late bands with sixteen that share a block
])
def test_shared_grammar(N, P, lens, n_max, forms):
    assert tuple(set(x.values()) for x in band_rule.choose(N, lens)) == forms
    d = synth.make_inputs("tiny", seed=4200 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=300)
    if n_max is not None:
        more = np.full((d["B"], n_max - d["n_max"], P), np.nan, dtype=np.float32)
        d["n_max"], d["log_emit"] = n_max, np.concatenate([d["log_emit"], more], axis=1)
    print("case", N, P, lens, n_max, flush=True)
    wl = bd.Workload(d)
    wl.workspace.fill_(255)  # nothing is read before it is written
    g = np.linspace(-1.0, 2.0, len(lens)).astype(np.float32)
    wl.forward_backward(torch.tensor(g, device="cuda:0"))
    many = len(lens) >= 60
    ref = oracle_batch_parallel(d, g) if many else O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"], g)
    check_all(wl.results(), ref)


def test_backward_twice_on_one_forward():
    """The exponents of partial sums lie where the pass has not written yet; none of it is needed by another reverse pass."""
    d = synth.make_inputs("tiny", seed=4299, pad_value=np.nan, N=65, P=20, B=3, lengths=[63, 17, 52], V=300)
    print("case two reverse passes", flush=True)
    wl = bd.Workload(d)
    wl.workspace.fill_(255)
    wl.forward()
    g = np.array([0.5, -1.0, 2.0], dtype=np.float32)
    for grad in (None, torch.tensor(g, device="cuda:0")):
        wl.backward(grad)
        check_all(wl.results(), O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"],
                                                  np.ones(3) if grad is None else g))


def test_one_grammar_per_sentence():
    d = synth.make_inputs_per_sentence("tiny", seed=4300, pad_value=np.nan, N=40, P=24, B=3, lengths=[50, 2, 61])
    print("case per-sentence bands", flush=True)
    wl = bd.Workload(d)
    wl.forward_backward(None)
    got = wl.results()
    for b in range(3):
        n = int(d["lengths"][b])
        lz, gL, gR, gr, ge = O.inside_backward_sentence(d["log_root"][b], d["L"][b], d["R"][b], d["log_emit"][b, :n], 1.0)
        check_logZ(got["logZ"][b:b + 1], np.array([lz]))
        for name, x, y in (("grad_L", got["grad_L"][b], gL), ("grad_R", got["grad_R"][b], gR),
                           ("grad_log_root", got["grad_log_root"][b], gr), ("grad_log_emit", got["grad_log_emit"][b, :n], ge)):
            check_grad(name, x, y)
