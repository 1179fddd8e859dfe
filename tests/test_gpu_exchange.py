"""The sum of a tile's partial products (finish_tile in csrc/gemm_nt_common.h) at every number of parts where its rounds change: two
parts, a last round of one to three, full rounds of four, both.  Launches of few rows on fp32 matrix instructions cut a tile into the
most parts; every case asserts how many it reaches.  Against the CPU oracle with the tolerances of tests/parity_util.py."""
import numpy as np
import pytest

from oracle import spcfg_oracle as O
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth
from parity_util import check_all

pytestmark = pytest.mark.gpu


def parts_of_tiles(N, P, lens):
    """Parts of the output tiles of all projection launches of a batch with at most 32 rows a width (32 x 128 tiles, K-steps of 32
    values, equal shares of at least two)."""
    up = lambda a, b: -(-a // b)
    Np, Pp, out = up(N, 64) * 64, up(P, 64) * 64, set()

    def launch(products):  # [(tiles, K-steps)], one after the other in the space that is shared out
        total = sum(t * k for t, k in products)
        share = up(total, min(128 if total < 1024 else 256 if total < 4096 else 512, max(1, total // 2)))
        u = 0
        for tiles, k in products:
            for _ in range(tiles):
                out.add((u + k - 1) // share - u // share + 1)
                u += k

    for w in range(1, max(lens)):
        c = [n - w + 1 for n in lens if n >= w]
        rows, pre, suf, mid = sum(c), len(c), sum(x >= 2 for x in c), sum(max(0, x - 2) for x in c)
        assert rows <= 32
        t = lambda r, cols: up(r, 32) * up(cols, 128)
        if w == 1:
            launch([(t(rows, 2 * Np), Pp // 32)])
            launch([(t(rows, P), Np // 16)])
            continue
        launch([(t(pre + mid, Np), Np // 32), (t(mid + suf, Np), Np // 32)] if Np % 128 == 0 else [(t(rows, 2 * Np), Np // 32)])
        parts = [(t(pre, Np), Np // 32), (t(mid, Np), Np // 16), (t(suf, Np), Np // 32)]
        launch(parts if up(rows, 32) * up(Np, 128) * (Np // 16) > sum(a * b for a, b in parts) else [(t(rows, Np), Np // 16)])
    return out


@pytest.mark.parametrize("N,P,lens,parts", [
    (64, 64, [5], {1, 2}),
    (130, 200, [9, 4], {3, 4, 6}),
    (300, 90, [11], {2, 5, 10}),
    (100, 430, [6, 5], {2, 4, 7}),
    (512, 512, [14, 9], {8, 16}),
    (700, 1100, [10], {9, 11, 15, 16}),
    (450, 1500, [8], {8, 11, 12, 16}),
    (1000, 64, [7], {1, 8, 16, 32}),
])
def test_parts(N, P, lens, parts):
    assert parts_of_tiles(N, P, lens) >= parts, parts_of_tiles(N, P, lens)
    d = synth.make_inputs("tiny", seed=6100 + N, pad_value=np.nan, N=N, P=P, B=len(lens), lengths=lens, V=90)
    print("case parts", N, P, lens, flush=True)
    wl = bd.Workload(d, flags=bd.FLAG_FP32_MFMA)
    wl.workspace.fill_(255)  # nothing is read before it is written
    wl.forward_backward(None)
    first = wl.results()
    check_all(first, O.inside_backward(d["log_root"], d["L"], d["R"], d["log_emit"], d["lengths"]))
    wl.forward_backward(None)
    for k, v in wl.results().items():
        assert np.array_equal(v, first[k]), f"{k}: two runs differ bitwise"
