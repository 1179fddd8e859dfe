"""The projection kernel for few rows (csrc/gemm_short.hip) at the edges of its tiles: fewer K-steps than wavefronts,
row and column remainders of every tile shape, prefix / middle / suffix parts, one grammar per sentence; every case asserts
the tiles that it reaches.  Against the CPU oracle, with the tolerances of tests/parity_util.py."""
import numpy as np
import pytest

import short_rule
from oracle import spcfg_oracle as O
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth
from parity_util import check_all, check_grad, check_logZ

pytestmark = pytest.mark.gpu


# fwd, bwd: tiles that the case has to reach (rows x columns, "p" in parts)
@pytest.mark.parametrize("N,P,lens,fwd,bwd", [
    (5, 70, [17, 16, 2], ["16x16"], ["16x16"]),          # one K-step pair: most wavefronts have none; one row over a tile
    (66, 130, [33, 3], ["16x16p"], ["16x16"]),           # remainders in rows, columns and K
    (190, 61, [20] * 5, ["16x16"], ["16x16"]),           # three blocks of 64 nonterminals: no parts forward
    (190, 61, [12] * 64, ["16x16", "32x16", "32x32", "64x32"], ["16x16p", "32x16p", "32x32p"]),  # the same, parts in reverse
    (512, 65, [19, 18, 12, 9, 17], ["16x16p", "32x16p"], ["16x16"]),  # parts forward
    (512, 300, [12] * 26, ["16x16p", "32x16p", "32x32p", "64x32p"], ["16x16p", "32x16p", "32x32p"]),  # parts in both directions
    (1000, 40, [9] * 30, ["16x16p", "32x16p", "32x32p", "64x32p"], ["16x16p", "32x16p", "32x32p"]),   # long K
    (1000, 40, [7] * 90, ["64x64p"], ["32x32p", "64x32p", "64x64p"]),  # the tallest tiles, with remainders, in parts
    (900, 40, [8] * 70, ["64x32", "64x64"], ["64x32p"]),  # and over all columns
])
def test_shared_grammar(N, P, lens, fwd, bwd):
    reached = short_rule.tiles(N, P, lens)
    assert reached[0] >= set(fwd) and reached[1] >= set(bwd), reached
    d = synth.make_inputs("tiny", seed=4000 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=300)
    print("case", N, P, lens, flush=True)
    wl = bd.Workload(d)
    wl.forward_backward(None)
    check_all(wl.results(), O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"]))


@pytest.mark.parametrize("N,P,lens,fwd,bwd", [
    (130, 50, [18, 2, 35], ["16x16"], ["16x16"]),
    (70, 200, [5] * 40, ["16x16", "32x32"], ["32x32"]),
    (600, 500, [33] * 6, ["32x32", "64x32"], ["32x16", "32x32"]),
])
def test_one_grammar_per_sentence(N, P, lens, fwd, bwd):
    reached = short_rule.tiles(N, P, lens, per_sentence=True)
    assert reached[0] >= set(fwd) and reached[1] >= set(bwd), reached
    d = synth.make_inputs_per_sentence("tiny", seed=4100 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens)
    print("case", N, P, lens, flush=True)
    wl = bd.Workload(d)
    wl.forward_backward(None)
    got = wl.results()
    for b in (0, 1, len(lens) - 1):
        n = int(d["lengths"][b])
        lz, gL, gR, gr, ge = O.inside_backward_sentence(d["log_root"][b], d["L"][b], d["R"][b], d["log_emit"][b, :n], 1.0)
        check_logZ(got["logZ"][b:b + 1], np.array([lz]))
        for name, x, y in (("grad_L", got["grad_L"][b], gL), ("grad_R", got["grad_R"][b], gR),
                           ("grad_log_root", got["grad_log_root"][b], gr), ("grad_log_emit", got["grad_log_emit"][b, :n], ge)):
            check_grad(name, x, y)
