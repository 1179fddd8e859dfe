"""Split-point sums of launches with few spans (k_split_fwd_few / k_split_bwd_few in csrc/kernels_elem.hip): the terms of a
span shared by the wavefronts of one workgroup.  Against the CPU oracle, with the tolerances of tests/parity_util.py: every
number of terms from 1 to 46 (all five shapes, with and without idle wavefronts), the last lanes of a block of nonterminals,
both forms within one pass, bands, one grammar per sentence."""
import numpy as np
import pytest

from oracle import spcfg_oracle as O
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth
from parity_util import check_all, check_grad, check_logZ

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,lens", [
    (30, 41, [47]),             # 1 to 46 terms, one workgroup a span
    (300, 20, [35, 2, 18]),     # the second block of nonterminals is nearly empty
    (65, 33, [66, 65, 3]),      # bands late: sums that go on from a partial one, with 0 to 6 terms
    (70, 30, [28] * 90),        # about 2400 spans in the shortest widths, 90 in the last: both forms
    (20, 10, [60] * 8),         # reverse widths 16 to 27 request too many rows and take the plain form, wider ones do not
    (1100, 12, [9, 4]),         # five blocks of nonterminals: the reverse sums stay in the plain form
])
def test_shared_grammar(N, P, lens):
    d = synth.make_inputs("tiny", seed=4400 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=300)
    print("case", N, P, lens[:3], len(lens), flush=True)
    wl = bd.Workload(d)
    wl.workspace.fill_(255)  # nothing is read before it is written
    wl.forward_backward(None)
    check_all(wl.results(), O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"]))
    first = wl.results()
    wl.forward_backward(None)
    for k, v in wl.results().items():
        assert np.array_equal(v, first[k]), f"{k}: two runs differ bitwise"


def test_one_grammar_per_sentence():
    d = synth.make_inputs_per_sentence("tiny", seed=4500, pad_value=np.nan, N=40, P=24, B=3, lengths=[40, 2, 21])
    print("case per-sentence few", flush=True)
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
