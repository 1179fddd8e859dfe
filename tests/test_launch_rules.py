"""In which form the products on bf16 planes run (csrc/gemm_forms.h), asked of the library's own host code on the CPU, against the
measured times of the forms."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.check_call([hipcc, "--cuda-host-only", "-O1", "-std=c++17", "-w", "-I", os.path.join(ROOT, "paper_2310_14997_amd", "csrc"),
                           "-x", "hip", os.path.join(ROOT, "tests", "host", "launch_rules.cpp"), "-o", exe])

    def run(lines):
        res = subprocess.run([exe], input="\n".join(lines) + "\n", stdout=subprocess.PIPE, text=True, timeout=60, check=True)
        return [[int(x) for x in line.split()] for line in res.stdout.splitlines()]
    return run


# ((planes, N, reverse, rows, prefix spans = suffix spans), us of every form: tile, "whole" tiles instead of equal shares, the reverse
# product as "one" instead of in parts, or tiles "staged" through registers).  Measured with the caches' contents replaced between launches.
PROJECTIONS = [
    ((1, 576, 1, 1984, 64), {"64x128 whole one": 13.6, "64x128 one": 18.7, "128x128 whole one": 19.9, "staged": 20.0,
      "64x128": 20.9, "32x128 one": 21.1, "128x128 one": 23.9, "128x256 whole one": 25.3, "128x128": 26.7, "32x128": 27.1}),
    ((1, 768, 1, 1984, 64), {"64x128 whole one": 15.9, "64x128 one": 20.5, "128x128 whole one": 22.5, "staged": 23.3,
      "32x128 one": 25.8, "64x128": 25.9, "128x256 whole one": 28.8, "128x128 one": 29.8, "128x128": 29.8, "32x128": 30.8}),
    ((1, 576, 0, 864, 32), {"32x128": 9.1, "64x128 whole": 10.4, "128x128 whole": 13.3, "staged": 16.9, "128x256 whole": 17.4,
      "128x128": 17.7, "64x128": 18.1}),
    ((1, 640, 1, 1984, 64), {"64x128 whole one": 15.5, "64x128 one": 19.6, "128x128 whole one": 21.3, "64x128": 21.7,
      "staged": 21.8, "32x128 one": 22.0, "128x128 one": 26.2, "128x256 whole one": 27.8, "32x128": 28.1, "128x128": 29.0}),
    ((1, 1024, 1, 1248, 32), {"64x128 whole one": 17.4, "64x128 one": 21.3, "64x128": 22.9, "128x128 whole one": 24.4,
      "staged": 24.7, "32x128 one": 26.2, "128x128 one": 30.5, "32x128": 31.3, "128x256 whole one": 32.2, "128x128": 32.6}),
    ((1, 64, 0, 1248, 32), {"64x128 whole": 7.4, "128x128 whole": 10.5, "128x256 whole": 12.2, "64x128": 12.5, "staged": 12.8,
      "32x128": 14.2}),
    ((1, 1024, 0, 1056, 32), {"64x128 whole": 13.1, "64x128": 13.9, "128x128 whole": 16.4, "32x128": 18.4,
      "128x256 whole": 21.7, "128x128": 22.0, "staged": 22.2}),
    ((1, 1088, 1, 1056, 32), {"64x128 whole one": 18.3, "64x128 one": 21.8, "64x128": 25.1, "staged": 25.4,
      "128x128 whole one": 25.8, "32x128 one": 26.0, "128x128": 30.6, "32x128": 30.7, "128x128 one": 30.7,
      "128x256 whole one": 34.5}),
    ((1, 1280, 0, 660, 20), {"64x128 whole": 14.1, "128x128 whole": 18.1, "64x128": 18.5, "staged": 22.6, "32x128": 23.4,
      "128x128": 24.5, "128x256 whole": 24.6}),
    ((1, 1088, 0, 660, 20), {"64x128 whole": 12.7, "128x128 whole": 16.5, "64x128": 18.0, "staged": 19.6, "32x128": 20.8,
      "128x256 whole": 22.2, "128x128": 24.7}),
    ((1, 512, 0, 1056, 32), {"32x128": 8.7, "64x128 whole": 9.9, "64x128": 12.6, "128x128 whole": 13.2, "staged": 14.1,
      "128x256 whole": 16.6}),
    ((1, 768, 0, 704, 32), {"32x128": 9.8, "64x128 whole": 11.2, "128x128 whole": 14.6, "staged": 15.6, "64x128": 16.4,
      "128x128": 18.0, "128x256 whole": 19.0}),
    ((1, 64, 0, 208, 8), {"64x128 whole": 7.4, "128x128 whole": 10.0, "128x256 whole": 12.0, "64x128": 12.2, "staged": 12.6,
      "32x128": 14.1}),
    ((1, 1280, 0, 10, 1), {"staged": 9.0, "64x128 whole": 9.6, "128x128 whole": 10.7, "32x128": 11.2, "64x128": 14.5,
      "128x256 whole": 16.2, "128x128": 19.2}),
    ((1, 1088, 0, 60, 3), {"staged": 11.6, "64x128 whole": 12.2, "32x128": 12.5, "128x128 whole": 13.8, "64x128": 15.6,
      "128x256 whole": 19.6, "128x128": 21.1}),
    ((1, 1280, 1, 38, 1), {"32x128": 14.2, "staged": 14.3, "32x128 one": 15.1, "64x128": 17.8, "64x128 whole one": 19.0,
      "128x128 whole one": 20.6, "64x128 one": 22.7, "128x128": 23.6, "128x256 whole one": 30.7}),
    ((1, 1024, 1, 38, 1), {"staged": 15.6, "64x128 whole one": 15.6, "32x128": 15.8, "32x128 one": 16.5,
      "128x128 whole one": 18.1, "64x128 one": 19.3, "64x128": 21.1, "128x256 whole one": 26.4, "128x128 one": 27.5,
      "128x128": 29.2}),
    ((1, 1280, 0, 38, 1), {"staged": 10.7, "32x128": 11.2, "64x128 whole": 12.4, "128x128 whole": 13.0, "64x128": 16.3,
      "128x256 whole": 19.3, "128x128": 21.2}),
    ((1, 1024, 0, 38, 1), {"64x128 whole": 10.5, "staged": 10.8, "32x128": 11.3, "128x128 whole": 11.5, "64x128": 14.2,
      "128x256 whole": 16.8, "128x128": 18.1}),
    ((1, 4096, 1, 1248, 32), {"128x256 whole one": 95.9, "128x256 one": 96.0, "128x256": 104.9, "128x128 one": 106.1,
      "64x128 one": 119.9, "128x128 whole one": 123.2, "staged": 124.3, "64x128 whole one": 128.9, "128x128": 131.1,
      "64x128": 155.9}),
    ((1, 2048, 0, 38, 1), {"32x128": 12.0, "64x128 whole": 14.0, "staged": 15.1, "128x128 whole": 16.1, "64x128": 16.5,
      "128x128": 21.1, "128x256 whole": 24.8}),
    ((1, 3072, 0, 1056, 32), {"128x256 whole": 46.4, "128x256": 54.2, "128x128 whole": 59.1, "128x128": 59.5,
      "64x128 whole": 64.9, "64x128": 66.0, "32x128": 91.8, "staged": 96.5}),
    ((1, 4096, 0, 1248, 32), {"128x256": 92.9, "128x128": 101.7, "128x256 whole": 108.7, "128x128 whole": 109.7,
      "staged": 118.4, "64x128": 121.3, "64x128 whole": 125.2, "32x128": 174.4}),
    ((1, 4096, 1, 48, 8), {"32x128 one": 20.2, "staged": 23.4, "64x128 one": 24.0, "32x128": 27.9, "64x128": 30.3,
      "128x128 one": 30.5, "64x128 whole one": 36.2, "128x128": 38.7}),
    ((2, 512, 0, 1984, 64), {"64x128 whole": 17.3, "128x128 whole": 19.6, "128x128": 21.6, "64x128": 22.0,
      "128x256 whole": 25.2, "32x128": 28.6, "128x256": 32.4}),
    ((2, 768, 0, 1248, 32), {"64x128 whole": 20.6, "128x128 whole": 23.9, "128x128": 24.1, "64x128": 25.4,
      "128x256 whole": 31.7, "32x128": 32.6, "128x256": 34.4}),
    ((2, 384, 0, 1984, 64), {"64x128 whole": 14.4, "128x128 whole": 17.4, "64x128": 19.5, "128x256 whole": 22.6, "32x128": 22.7,
      "128x128": 23.3, "128x256": 31.1}),
    ((2, 576, 0, 1984, 64), {"128x128 whole": 20.6, "64x128": 25.6, "128x128": 26.7, "128x256 whole": 27.2,
      "64x128 whole": 30.1, "128x256": 31.6, "32x128": 32.3}),
    ((2, 1024, 0, 704, 32), {"64x128 whole": 19.9, "64x128": 24.9, "128x128 whole": 25.3, "32x128": 29.6, "128x128": 30.3,
      "128x256 whole": 36.0}),
    ((2, 320, 0, 1984, 64), {"64x128 whole": 13.0, "128x128 whole": 15.9, "64x128": 17.7, "32x128": 18.9, "128x256 whole": 20.7,
      "128x128": 21.0}),
    ((2, 3072, 0, 1056, 32), {"128x256 whole": 106.2, "128x256": 112.3, "128x128": 123.2, "128x128 whole": 135.7,
      "64x128 whole": 156.6, "64x128": 156.7}),
    ((2, 64, 0, 208, 8), {"32x128": 7.0, "64x128 whole": 8.1, "64x128": 8.3, "128x128 whole": 11.0, "128x128": 11.1,
      "128x256": 13.6, "128x256 whole": 13.6}),
    ((2, 1024, 0, 38, 1), {"32x128": 13.3, "64x128 whole": 18.3, "128x128 whole": 19.6, "64x128": 20.7, "128x128": 28.2}),
    ((2, 1088, 0, 60, 3), {"32x128": 16.8, "64x128": 20.0, "64x128 whole": 20.2, "128x128 whole": 24.1, "128x128": 26.8,
      "128x256 whole": 36.3}),
    ((2, 1280, 0, 38, 1), {"32x128": 15.1, "64x128": 18.1, "64x128 whole": 22.4, "128x128": 23.3, "128x128 whole": 24.5}),
    ((2, 1280, 0, 10, 1), {"32x128": 13.0, "64x128": 16.3, "64x128 whole": 19.7, "128x128": 21.0, "128x128 whole": 21.0}),
    ((2, 2048, 0, 38, 1), {"32x128": 15.9, "64x128": 19.8, "128x128": 25.1, "64x128 whole": 28.6, "128x128 whole": 32.1}),
    ((2, 4096, 0, 1248, 32), {"128x256": 221.7, "128x128": 247.1, "128x256 whole": 268.0, "128x128 whole": 269.7,
      "64x128": 301.6, "64x128 whole": 312.4, "32x128": 443.7}),
]


def test_projection_forms(ask):
    forms = ask("nt %d %d %d %d %d %d" % (*case, case[4]) for case, _ in PROJECTIONS)
    slow = []
    for (case, times), (bm, bn, whole, parts) in zip(PROJECTIONS, forms):
        name = "staged" if bm == 0 else "%dx%d" % (bm, bn) + (" whole" if whole else "") + (" one" if case[2] and not parts else "")
        # (forms within 15 % of each other are as close as the estimate can tell apart)
        if not times.get(name, 1e9) <= 1.15 * min(times.values()):
            slow.append((case, name, times))
    assert not slow, slow


# (output tiles, steps, us in equal shares, us in whole tiles) of rule-gradient products on one plane
RULE_GRADIENTS = [
    (3, 6, 19.4, 11.1), (3, 60, 34.8, 42.4), (16, 390, 75.2, 236.5), (64, 20, 28.4, 21.2), (64, 60, 36.3, 44.3),
    (144, 20, 33.0, 22.9), (144, 390, 224.6, 264.6), (196, 60, 64.0, 54.4), (196, 390, 296.5, 344.2), (240, 150, 149.8, 135.9),
    (256, 150, 141.9, 141.9), (297, 60, 84.8, 102.4), (297, 150, 176.7, 235.5), (297, 390, 451.9, 668.4),
    (306, 390, 473.9, 679.3), (324, 150, 194.1, 235.2), (324, 390, 497.8, 674.8), (400, 20, 51.8, 47.2), (400, 390, 625.6, 716.9),
    (540, 150, 312.4, 373.7), (540, 390, 823.6, 1037.4), (576, 60, 147.2, 164.4), (784, 150, 446.4, 510.4), (1024, 6, 54.7, 52.5),
]


def test_rule_gradient_shares(ask):
    shares = ask("tn %d %d" % (tiles, steps) for tiles, steps, _, _ in RULE_GRADIENTS)
    for (tiles, steps, cut, whole), (share,) in zip(RULE_GRADIENTS, shares):
        got = whole if share == steps else cut
        assert got <= 1.1 * min(cut, whole), (tiles, steps, share, cut, whole)
        if share != steps:  # at most a workgroup per CU, none without work
            assert -(-tiles * steps // share) <= 256 and share >= 2
