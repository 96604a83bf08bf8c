"""GPU parity of what a call takes to the device: sets of one segment inline and
of several in tables, delay tables shared by the calls of a distribution, more
distributions than the context keeps tables for."""
import pytest

from gpu_util import compare_all
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu


def _syn(mean, sd=0.75):
    return {"weight": W.W_E, "delay": {"kind": "normal", "mean": mean, "sd": sd, "lo": 0.1}}


RULES = [{"rule": "fixed_indegree", "n": 7}, {"rule": "fixed_indegree", "n": 7, "multapses": False},
         {"rule": "fixed_outdegree", "n": 5}, {"rule": "fixed_outdegree", "n": 5, "multapses": False},
         {"rule": "fixed_total_number", "n": 300}, {"rule": "fixed_total_number", "n": 300, "autapses": False},
         {"rule": "fixed_total_number", "n": 90, "multapses": False}, {"rule": "pairwise_bernoulli", "p": 0.2}]


@pytest.mark.parametrize("rule", RULES, ids=lambda r: r["rule"])
@pytest.mark.parametrize("policy", [None, (1, 1, 1.0)])
def test_segments_and_distributions(rule, policy):
    one, two, far = [(0, 20, 40)], [(0, 70, 30), (0, 0, 15)], [(1, 5, 25)]
    conn = {"autapses": True, "multapses": True, **rule}
    calls = [(s, t, conn, _syn(m), -1) for m in (1.5, 2.0) for s, t in
             ((one, one), (two, one), (one, two), (two, two), (far, one), (far + one, two), (one, far))]
    script = {"name": "tables", "P": 2, "seed": 9, "dt": 0.1,
              "ops": [("create", 0, 100), ("create", 1, 40)] + [("connect",) + cl for cl in calls]}
    if policy is not None:
        script["map_policy"] = policy
    for host in (0, 1):
        compare_all(script, host)


def test_more_distributions_than_tables():
    conn = {"rule": "fixed_indegree", "n": 1, "autapses": True, "multapses": True}
    s = [(0, 0, 3)]
    ops = [("create", 0, 3)] + [("connect", s, s, conn, _syn(1.0 + (k % 4100) * 1e-3), -1) for k in range(4200)]
    assert compare_all({"name": "distributions", "P": 1, "seed": 2, "dt": 0.1, "ops": ops}, 0) == 3 * 4200
