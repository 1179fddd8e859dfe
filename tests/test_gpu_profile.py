"""The profile's launches and bytes of the split-point sums are those of the kernels that ran, with and without bands."""
import numpy as np
import pytest
import torch

import band_rule
from paper_2310_14997_amd import binding as bd
from paper_2310_14997_amd import synth

pytestmark = pytest.mark.gpu


def rows_moved(N, lens, n_max):
    """Chart rows that the split launches read and write, counted span by span and tile by tile: (forward, reverse)."""
    fwd, bwd = band_rule.choose(N, lens)
    W, f, r = band_rule.W, 0, 0
    for n in lens:
        for w in range(2, n + 1):
            w0 = w // W * W
            for i in range(n - w + 1):
                if w0 in fwd:  # two children rows for every term with a child inside the band; the partial sum twice written
                    f += 3 + 2 * sum(1 for k in range(1, w) if k >= w0 or w - k >= w0)
                else:
                    f += 1 + 2 * (w - 1)
        for w0 in fwd:
            for i0 in range(0, n - w0 + 1, W):
                f += (2 * W + W - 1) * len([s for s in range(i0 + 1, n) if any(i < s < i + w0 for i in range(i0, i0 + W))])
        for w in range(1, n):
            w0, wt = w // W * W, w // W * W + W
            for i in range(n - w + 1):
                parents = [j - i for j in range(i + w + 1, n + 1)] + [i + w - a for a in range(i)]
                if w0 in bwd:  # both halves of the sum written, read and written again
                    r += 6 + 2 * sum(1 for v in parents if v < wt)
                else:
                    r += 2 + 2 * len(parents)
        for w0 in bwd:
            for i0 in range(0, n - w0 + 1, W):
                r += (2 * W + W - 1) * (max(0, n - i0 - w0 - W + 1) + i0 + W - 1)
    return f, r


@pytest.mark.parametrize("N,P,lens,n_max", [
    (30, 10, [9, 4], 9),
    (7, 9, [52, 51, 50, 53], 60),
    (180, 12, [60] * 70, 60),
])
def test_launches_and_bytes_of_the_split_sums(N, P, lens, n_max):
    d = synth.make_inputs("tiny", seed=4600 + N, N=N, P=P, B=len(lens), lengths=lens, V=50)
    if n_max > d["n_max"]:
        d["log_emit"] = np.concatenate([d["log_emit"], np.zeros((d["B"], n_max - d["n_max"], P), np.float32)], axis=1)
        d["n_max"] = n_max
    print("case profile", N, len(lens), flush=True)
    wl = bd.Workload(d)
    bd.spcfg_profile_enable(True)
    wl.forward_backward()
    torch.cuda.synchronize()
    prof = bd.spcfg_profile_read()
    bd.spcfg_profile_enable(False)
    fwd, bwd = band_rule.choose(N, lens)
    assert prof["split_fwd"]["launches"] == max(lens) - 1 + len(fwd)
    assert prof["split_bwd"]["launches"] == min(max(lens), n_max - 1) + len(bwd)
    assert (prof["setup"]["launches"], prof["root"]["launches"], prof["gemm_grad"]["launches"]) == (4, 4, 5)
    f, r = rows_moved(N, lens, n_max)
    assert prof["split_fwd"]["work"] == 4 * N * f
    assert prof["split_bwd"]["work"] == 4 * N * r


@pytest.mark.parametrize("N,P,lens,all_shared", [(30, 10, [9, 4], True), (1024, 600, [9, 4], False)])
def test_shared_launches_are_kept_apart(N, P, lens, all_shared):
    d = synth.make_inputs("tiny", seed=4700 + N, N=N, P=P, B=len(lens), lengths=lens, V=50)
    print("case shared launches", N, len(lens), flush=True)
    wl = bd.Workload(d)
    wl.forward_backward()
    torch.cuda.synchronize()
    bd.spcfg_profile_enable(True)
    wl.forward_backward()
    torch.cuda.synchronize()
    prof, shared = bd.spcfg_profile_read(), bd.spcfg_profile_read_shared()
    for product, sums in (("gemm_fwd", "split_fwd"), ("gemm_bwd", "split_bwd")):
        assert shared[product]["launches"] == shared[sums]["launches"] and shared[product]["ms"] == shared[sums]["ms"]
        # a small grammar's sums all come with a product, but the reverse pass's first; a large one's none
        assert prof[sums]["launches"] - shared[sums]["launches"] == ((sums == "split_bwd") if all_shared else prof[sums]["launches"])
        for c in (product, sums):
            for key in ("ms", "work"):
                assert (shared[c][key] > 0) == all_shared and shared[c][key] <= prof[c][key]
    assert all(not any(shared[c].values()) for c in ("setup", "root", "gemm_grad"))
    bd.spcfg_profile_enable(False)


def test_bytes_of_the_set_up():
    N, P = 30, 10
    d = synth.make_inputs("tiny", seed=4800, N=N, P=P, B=2, lengths=[9, 4], V=50)
    print("case set-up bytes", flush=True)
    wl = bd.Workload(d)
    bd.spcfg_profile_enable(True)
    # scoring: L and R read, the forward panels written; the reverse pass writes its own
    tokens = int(np.sum(d["lengths"]))
    wl.forward()
    torch.cuda.synchronize()
    assert bd.spcfg_profile_read()["setup"]["work"] == 4 * 2 * N * (N + P) * 2 + 8 * tokens * P
    wl.backward()
    torch.cuda.synchronize()
    assert bd.spcfg_profile_read()["setup"]["work"] == 4 * 2 * N * (N + P) * 2
    wl.forward_backward()
    torch.cuda.synchronize()
    assert bd.spcfg_profile_read()["setup"]["work"] == 4 * 2 * N * (N + P) * 3 + 8 * tokens * P
    bd.spcfg_profile_enable(False)
