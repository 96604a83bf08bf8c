"""GPU parity of the first-index array where long runs of sources have no
connections (before, between and after the used ones), on both ways of
building it and in the image-numbering pass."""
import pytest

from gpu_util import compare_all

pytestmark = pytest.mark.gpu

SYN = {"weight": {"kind": "const", "mean": 0.5}, "delay": {"kind": "const", "mean": 1.5}}


def _script(P, first, used, last, K, n_tgt):
    """used sources between first and last unused ones on host 0, targets with in-degree K; host 1 adds remote sources"""
    n = first + used + last
    ops = [("create", 0, n), ("create", 0, n_tgt)]
    if P > 1:
        ops.append(("create", 1, 50))
    tgt = [(0, n, n_tgt)]
    conn = {"rule": "fixed_indegree", "n": K, "autapses": True, "multapses": True}
    ops.append(("connect", [(0, first, used)], tgt, conn, SYN, -1))
    if P > 1:
        ops.append(("connect", [(1, 10, 30)], tgt, conn, SYN, -1))
    return {"name": f"rows {first}+{used}+{last} K={K}", "P": P, "seed": 5, "dt": 0.1, "ops": ops}


@pytest.mark.parametrize("P", [1, 2])
@pytest.mark.parametrize("first,used,last", [(0, 1, 0), (7, 3, 8), (9, 2, 9), (700, 1, 0), (0, 1, 700), (513, 40, 1021)])
@pytest.mark.parametrize("K,n_tgt", [(1, 3), (30, 70)])
def test_row_gaps(P, first, used, last, K, n_tgt):
    assert compare_all(_script(P, first, used, last, K, n_tgt), 0) == K * n_tgt * P
