"""Products of the bf16 mode at the sizes where their tiles change (csrc/gemm_nt3.hip, csrc/gemm_tn3.hip): rows that fill, cross and
miss 32-, 64- and 128-row tiles, columns that end inside a 128- and a 256-wide tile, K with and without whole steps, reductions that
end inside a step, parts and no parts.  Against the fp32 mode of the same library, which the oracle checks elsewhere: operands
rounded to 2^-9 give gradients within 1e-2 (relative 2-norm), log Z within 2e-3 with single operands and 1e-4 with two pieces."""
import numpy as np
import pytest

from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,lens", [
    (64, 65, [5, 2]),                  # one step of K, one tile, a reduction far below a step
    (130, 400, [20] * 9),              # three 64-column blocks: no parts, columns end inside every tile shape
    (512, 200, [12] * 33),             # rows from 33 to 363: short tiles, whole and cut
    (640, 1000, [10] * 120),           # 128-row tiles, 2.5 of 256 columns
    (1024, 96, [14] * 64),             # both tall shapes
])
def test_against_fp32(N, P, lens):
    d = synth.make_inputs("tiny", seed=5300 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=60)
    print("case bf16 tiles", N, P, len(lens), flush=True)
    ref = bd.Workload(d)
    ref.forward_backward(None)
    ref = ref.results()
    for flags, bar in ((0, 1e-4), (bd.FLAG_BF16_SINGLE_FORWARD, 2e-3)):
        wl = bd.Workload(d, precision=bd.PRECISION_BF16, flags=flags)
        wl.workspace.fill_(255)  # nothing is read before it is written
        wl.forward_backward(None)
        got = wl.results()
        assert np.all(np.abs(got["logZ"] - ref["logZ"]) <= bar * np.abs(ref["logZ"]))
        for k in ("grad_L", "grad_R", "grad_log_root", "grad_log_emit"):
            assert np.linalg.norm(got[k] - ref[k]) <= 1e-2 * np.linalg.norm(ref[k]), (flags, k)
        wl.forward_backward(None)
        for k, v in wl.results().items():
            assert np.array_equal(v, got[k]), f"{k}: two runs differ bitwise"
