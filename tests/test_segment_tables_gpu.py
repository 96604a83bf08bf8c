"""GPU parity of keys in target order around the number of source segments whose
addends fit beside the digit histograms: two 8-bit digits take 2 KB of 26, and a
segment 8 B."""
import pytest

from gpu_util import compare_all
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu

SYN = {"weight": W.W_E, "delay": {"kind": "normal", "mean": 1.5, "sd": 0.75, "lo": 0.1}}


@pytest.mark.parametrize("n_seg", [2047, 2048, 2049, 3071, 3072, 3073, 3500])
@pytest.mark.parametrize("equal", [True, False])
def test_segments_around_the_limit(n_seg, equal):
    sizes = [1] * n_seg if equal else [2] + [1] * (n_seg - 1)
    src, at = [], 0
    for m in sizes:
        src.append((0, at, m))
        at += m
    src.reverse()
    conn = {"rule": "fixed_indegree", "n": 300, "autapses": True, "multapses": True}
    ops = [("create", 0, at), ("connect", src, [(0, 5, 40)], conn, SYN, -1)]
    assert compare_all({"name": f"{n_seg} segments", "P": 1, "seed": 6, "dt": 0.1, "ops": ops}, 0) == 300 * 40
