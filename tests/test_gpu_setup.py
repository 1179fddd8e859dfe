"""Set-up and root kernels at the sizes where their forms change (csrc/kernels_elem.hip), and the panels that a call packs
(csrc/spcfg_api.hip): against the CPU oracle with the tolerances of tests/parity_util.py; one call against two bit for bit."""
import numpy as np
import pytest
import torch

from oracle import spcfg_oracle as O
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth
from parity_util import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,lens", [
    (6, 4099, [4, 2]),          # emission rows past the values that a workgroup keeps, with a ragged end and odd addresses
    (5, 4160, [3]),             # the same with whole 16-byte loads
    (2051, 5, [3, 2]),          # root scores past the values that a workgroup keeps
    (3, 4, [2, 5, 3] * 100),    # sentences in several wavefronts of the span plan, not a multiple of four or 64
    (2, 3, [2] * 957 + [6, 2, 4]),  # the most sentences
])
def test_sizes_at_which_the_kernels_change(N, P, lens):
    d = synth.make_inputs("tiny", seed=5100 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=60)
    print("case setup", N, P, len(lens), flush=True)
    wl = bd.Workload(d)
    wl.workspace.fill_(255)  # nothing is read before it is written
    wl.forward_backward(None)
    check_all(wl.results(), O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"]))


@pytest.mark.parametrize("N,P,lens,more,kw", [
    (30, 70, [9, 4, 2], 2, {}),                                   # fp32 panels only; n_max past the longest sentence
    (512, 300, [24] * 24, 0, {}),                                 # short and long launches
    (1024, 1024, [12] * 64, 0, {}),                               # launches on operand planes among them
    (1024, 1024, [12] * 64, 0, {"fp32_mfma": True}),
    (200, 100, [14, 9, 3], 1, {"precision": bd.PRECISION_BF16}),
    (200, 100, [14, 9, 3], 0, {"precision": bd.PRECISION_BF16, "bf16_single": True}),
])
def test_forward_then_reverse_is_the_one_call(N, P, lens, more, kw):
    d = synth.make_inputs("tiny", seed=5200 + N, N=N, P=P, B=len(lens), lengths=lens, V=60)
    if more:
        d["log_emit"] = np.concatenate([d["log_emit"], np.zeros((d["B"], more, P), np.float32)], axis=1)
        d["n_max"] += more
    print("case panels", N, P, kw, flush=True)
    flags = (bd.FLAG_FP32_MFMA if kw.get("fp32_mfma") else 0) | (bd.FLAG_BF16_SINGLE_FORWARD if kw.get("bf16_single") else 0)
    wl = bd.Workload(d, precision=kw.get("precision", bd.PRECISION_FP32), flags=flags)
    wl.workspace.fill_(255)
    wl.forward_backward(None)
    one = wl.results()
    wl.workspace.fill_(255)
    wl.forward()
    wl.backward()
    torch.cuda.synchronize()
    for k, v in wl.results().items():
        assert np.array_equal(v, one[k]), k
