"""The front-end's register-held rows and emission tiles at the sizes where they can go wrong: remainders of a tile, rows
that allow no 16-byte loads, rows past every register form, more positions than one segment."""
import numpy as np
import pytest

from oracle import rules_oracle as RO
from paper_2310_14997_amd import synth
from parity_util import check_grad
from test_gpu_rules import BWD_RTOL, FWD_RTOL, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(N=1, P=1, V=1, B=1, lengths=[1]),                                # one tile, nearly all of it past the end
    dict(N=3, P=65, V=129, B=3, lengths=[7, 0, 4]),                       # one row and one column over; an empty sentence
    dict(N=30, P=64, V=128, B=2, lengths=[5, 3]),                         # exactly one tile, 16-byte loads
    dict(N=60, P=70, V=257, B=40, lengths=[60 - b for b in range(40)]),   # 2400 positions: three segments, many repeats
    dict(N=9, P=4093, V=300, B=2, lengths=[6, 2]),                        # rows of 4102: eight 4-byte groups a thread
    dict(N=8, P=8188, V=40, B=2, lengths=[6, 2]),                         # rows of 8196: read in passes backward
    dict(N=5, P=33, V=16388, B=1, lengths=[3]),                           # vocabulary rows read in passes
    dict(N=5, P=33, V=16381, B=30, lengths=[40] * 30),                    # last register form, 4-byte loads
], ids=lambda k: "x".join(str(k[x]) for x in ("N", "P", "V", "B")))
def test_rows_and_tiles_at_their_edges(kw):
    print("case rules tiles", {k: kw[k] for k in "NPVB"}, flush=True)
    d = synth.make_logits("tiny", **kw)
    ref = RO.forward(d["root_logits"], d["L_logits"], d["R_logits"], d["emis_logits"], d["tokens"], d["lengths"])
    rng = np.random.default_rng(7)
    grads = {"grad_" + k: rng.normal(size=ref[k].shape).astype(np.float32) for k in ("log_root", "L", "R", "log_emit")}
    for b, n in enumerate(d["lengths"]):
        grads["grad_log_emit"][b, int(n):] = np.nan  # positions past a sentence's end are never read
    got, _, _ = run_gpu(d, grads)
    grads["grad_log_emit"] = np.nan_to_num(grads["grad_log_emit"])
    rb = RO.backward(d["root_logits"], d["L_logits"], d["R_logits"], d["emis_logits"], d["tokens"], d["lengths"], **grads)
    for k in ("log_root", "L", "R", "log_emit"):
        check_grad(k, got[k], ref[k], FWD_RTOL)
    for k in ("grad_root_logits", "grad_L_logits", "grad_R_logits", "grad_emis_logits"):
        check_grad(k, got[k], rb[k], BWD_RTOL)
