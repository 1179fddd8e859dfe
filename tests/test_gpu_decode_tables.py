"""Tree decoding at the sizes where its tables leave LDS: three of them fit up to n_max = 73, two up to 90, none above."""
import numpy as np
import pytest

from oracle import decode_oracle as D
from test_gpu_decode import decode_on_gpu, to_oracle_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [[2], [3, 2], [73, 2, 64, 65], [74, 73, 2], [91, 74]])
def test_trees_are_bit_exact_wherever_the_tables_lie(lengths):
    """Scores on a 1/64 grid: every fp32 sum is exact, so decisions and scores agree with the oracle bit for bit."""
    rng = np.random.default_rng(99 + sum(lengths))
    B, n_max = len(lengths), max(lengths)
    mu = rng.integers(0, 65, size=(B, n_max, n_max)).astype(np.float64) / 64.0
    print("case decode tables", lengths, flush=True)
    spans, score = decode_on_gpu(mu, lengths)
    for b, n in enumerate(lengths):
        ref_score, ref_spans = D.mbr_decode(to_oracle_layout(mu[b], n), n)
        assert [tuple(x) for x in spans[b, : n - 1]] == ref_spans, f"sentence {b} (n={n})"
        assert score[b] == ref_score
        assert np.all(spans[b, n - 1:] == -1)
