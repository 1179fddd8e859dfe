"""The products of the bf16 mode in the forms that csrc/gemm_forms.h can give them: tiles staged through registers and on planes, whole and
in shares, reverse products in parts and as one, rule gradients of more than 256 output tiles with a last round that is partly filled.
Every block of 64 rows and of 64 columns is held against the fp32 mode of the same library, which the oracle checks elsewhere: operands
rounded to 2^-9 give gradients within 1e-2 (relative 2-norm), every block too, so that a wrong tile shows wherever it lies;
log Z within 2e-3 with single operands and 1e-4 with two pieces."""
import numpy as np
import pytest

from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth

pytestmark = pytest.mark.gpu


def blocks_off(got, ref):
    """Largest relative 2-norm of the difference over blocks of 64 rows and of 64 columns."""
    worst = 0.0
    for g, r in ((got, ref), (got.T, ref.T)):
        for i in range(0, r.shape[0], 64):
            n = np.linalg.norm(r[i:i + 64])
            worst = max(worst, np.linalg.norm(g[i:i + 64] - r[i:i + 64]) / n if n > 0 else np.linalg.norm(g[i:i + 64]))
    return worst


@pytest.mark.parametrize("N,P,lens", [
    (200, 64, [12] * 100),        # whole 64-row tiles in parts, staged tiles, columns that end inside a tile
    (576, 100, [8] * 240),        # one product and parts, both whole: no whole number of 128-column blocks
    (1088, 130, [6, 5, 7] * 12),  # whole tiles next to staged ones
    (1300, 70, [7] * 100),        # tiles of 32 rows in shares next to whole ones of 64
    (2048, 2048, [8] * 12),       # rule gradients whose tiles run in blocks of 8 x 8
    (2112, 2112, [20] * 14),      # rule gradients in 297 tiles, equal shares that go on from tile to tile
    (2112, 2112, [3] * 8),        # the same, a reduction of one step: whole tiles
    (2200, 300, [9] * 24),        # 315 tiles, and 70 for the preterminals, whose last ones have 44 columns
])
def test_every_block(N, P, lens):
    d = synth.make_inputs("tiny", seed=6200 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=60)
    print("case bf16 forms", N, P, len(lens), flush=True)
    ref = bd.Workload(d)
    ref.forward_backward(None)
    ref = ref.results()
    for flags, bar in ((0, 1e-4), (bd.FLAG_BF16_SINGLE_FORWARD, 2e-3)):
        wl = bd.Workload(d, precision=bd.PRECISION_BF16, flags=flags)
        wl.workspace.fill_(255)  # nothing is read before it is written
        wl.forward_backward(None)
        got = wl.results()
        assert np.all(np.abs(got["logZ"] - ref["logZ"]) <= bar * np.abs(ref["logZ"]))
        for k in ("grad_L", "grad_R"):
            off = blocks_off(got[k], ref[k])
            print(k, flags, "%.1e" % off, flush=True)
            assert off <= 1e-2, (flags, k, off)
        for k in ("grad_L", "grad_R", "grad_log_root", "grad_log_emit"):
            assert np.linalg.norm(got[k] - ref[k]) <= 1e-2 * np.linalg.norm(ref[k]), (flags, k)
        wl.forward_backward(None)
        for k, v in wl.results().items():
            assert np.array_equal(v, got[k]), f"{k}: two runs differ bitwise"
