"""GPU parity of Prepare where the keys are written in target-major order
(every call a fixed in-degree or one-to-one rule) and at the edges of that
rule: runs around its shortest average length, one wave's unit of 2048
positions, targets covered by different calls, several segments, a single
source (no sorted bit), an assigned or out-degree call that rules it out."""
import pytest

from gpu_util import compare_all
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu

SYN = {"weight": W.W_E, "delay": {"kind": "normal", "mean": 1.5, "sd": 0.75, "lo": 0.1}}
SYN_C = {"weight": {"kind": "const", "mean": 0.25}, "delay": {"kind": "const", "mean": 0.3}}


def _in(K, **kw):
    return {"rule": "fixed_indegree", "n": K, "autapses": True, "multapses": True, **kw}


def _script(name, P, creates, calls, **kw):
    ops = [("create", h, n) for h, n in creates] + [("connect", s, t, c, y, a) for s, t, c, y, a in calls]
    return {"name": name, "P": P, "seed": 11, "dt": 0.1, "ops": ops, **kw}


@pytest.mark.parametrize("K", [1, 15, 16, 17, 63, 64, 65, 257, 2047, 2048, 2049, 5000])
@pytest.mark.parametrize("n_tgt", [1, 37])
def test_run_lengths(K, n_tgt):
    s = _script(f"runs K={K}", 1, [(0, 300), (0, n_tgt)], [([(0, 0, 300)], [(0, 300, n_tgt)], _in(K), SYN, -1)])
    assert compare_all(s, 0) == K * n_tgt


@pytest.mark.parametrize("policy", [None, (0, 2, 1.0), (1, 1, 1.0)])
@pytest.mark.parametrize("alpha", [-1, 0])
def test_calls_over_different_targets(policy, alpha):
    """Targets in no, one or several calls; segments out of order; Floyd and one-to-one runs; remote sources."""
    calls = [([(0, 0, 200)], [(0, 250, 40), (0, 10, 30)], _in(70), SYN, alpha),
             ([(1, 5, 90)], [(0, 0, 300)], _in(33), SYN_C, alpha),
             ([(0, 0, 300), (1, 0, 100)], [(0, 20, 100)], _in(129, autapses=False), SYN, alpha),
             ([(1, 50, 50), (0, 100, 50)], [(0, 270, 30)], _in(40, multapses=False), SYN, alpha),
             ([(0, 0, 60)], [(0, 30, 60)], {"rule": "one_to_one", "autapses": False}, SYN, alpha),
             ([(1, 0, 20)], [(1, 0, 20)], _in(9), SYN, alpha)]
    kw = {} if policy is None else {"map_policy": policy}
    for host in (0, 1):
        compare_all(_script("different targets", 2, [(0, 300), (1, 100)], calls, **kw), host)


@pytest.mark.parametrize("extra", [{"rule": "fixed_outdegree", "n": 3}, {"rule": "pairwise_bernoulli", "p": 0.2}])
def test_other_rules_keep_the_general_order(extra):
    calls = [([(0, 0, 50)], [(0, 0, 50)], _in(40), SYN, -1), ([(0, 0, 50)], [(0, 0, 50)], extra, SYN, -1)]
    compare_all(_script("mixed rules", 1, [(0, 50)], calls), 0)


def test_single_neuron():
    compare_all(_script("one neuron", 1, [(0, 1)], [([(0, 0, 1)], [(0, 0, 1)], _in(5000), SYN, -1)]), 0)


@pytest.mark.parametrize("variant,mode", [(1, 0), (6, 0), (12, 0), (0, 1), (3, 1)])
def test_sort_settings(variant, mode):
    s = W.balanced_collective(P=5, n_e=160, n_i=40, k_e=90, k_i=22)
    s["tune"] = {"sort_variant": variant, "sort_mode": mode}
    compare_all(s, 2)


@pytest.mark.parametrize("n_e", [1, 2007, 2008, 2009, 4057])
def test_group_ranges(n_e):
    """H/I ranges below, at and above the 2,048 entries a workgroup takes at a time (40 more by the inhibitory one)."""
    compare_all(W.balanced_collective(P=5, n_e=n_e, n_i=40, k_e=3, k_i=2), 3)


@pytest.mark.parametrize("sizes", [[50], [50, 30], [30, 30], [40, 40, 40], [40, 41, 39], [3] * 2049, [2] * 900 + [3] * 900])
@pytest.mark.parametrize("K", [63, 300])
def test_source_segments(sizes, K):
    """One, two, several source segments of equal and unequal length, more of them than fit beside the histograms."""
    n = sum(sizes)
    first = [sum(sizes[k + 1:]) for k in range(len(sizes))]         # the segments in descending order of neurons
    src = [(0, f, m) for f, m in zip(first, sizes)]
    half = src[: max(1, len(src) // 2)]
    calls = [(src, [(0, 5, 40)], _in(K), SYN, -1), (half, [(0, 0, 30)], _in(17), SYN_C, -1)]
    compare_all(_script(f"{len(sizes)} segments", 1, [(0, max(n, 50))], calls), 0)
