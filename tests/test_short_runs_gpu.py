"""GPU parity of generation over many short runs of units (node sets of several
hundred segments of one to a few neurons): tiles that meet one, two, many runs,
in calls of their own and in batches, where short calls and calls of short runs
take another launch than the others."""
import pytest

from gpu_util import GEN_ARRAYS, compare, compare_all, log
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu

SYN = {"weight": W.W_E, "delay": {"kind": "normal", "mean": 1.5, "sd": 0.75, "lo": 0.1}}
SYN_C = {"weight": {"kind": "const", "mean": 0.25}, "delay": {"kind": "const", "mean": 0.3}}
N = 6000


def _singles(n, first=0, step=3):
    return [(0, first + i * step, 1) for i in range(n)]


def _conn(rule, **kw):
    return {"rule": rule, "autapses": True, "multapses": True, **kw}


ALL = [(0, 0, N)]
MIXED = [(0, 0, 700)] + _singles(300, 1000) + [(0, 3000, 2000)] + _singles(200, 5000, 2)   # long runs around short ones
CALLS = {
    "indegree": lambda segs: (ALL, segs, _conn("fixed_indegree", n=3)),
    "indegree_no_autapses": lambda segs: (ALL, segs, _conn("fixed_indegree", n=3, autapses=False)),
    "indegree_long": lambda segs: (ALL, segs, _conn("fixed_indegree", n=300)),
    "floyd": lambda segs: (ALL, segs, _conn("fixed_indegree", n=5, multapses=False)),
    "floyd_larger": lambda segs: (ALL, segs, _conn("fixed_indegree", n=40, multapses=False)),
    "outdegree": lambda segs: (segs, ALL, _conn("fixed_outdegree", n=4)),
    "one_to_one": lambda segs: (segs, list(reversed(segs)), _conn("one_to_one")),
    "one_to_one_no_autapses": lambda segs: (segs, segs[1:] + segs[:1] if len({s[2] for s in segs}) == 1 else segs,
                                            _conn("one_to_one", autapses=False)),
}
SEGS = {"two": [(0, 5, 100), (0, 300, 40)], "singles": _singles(500), "mixed": MIXED, "three": [(0, 0, 600), (0, 700, 1), (0, 900, 600)]}


@pytest.mark.parametrize("segs", SEGS)
@pytest.mark.parametrize("call", CALLS)
def test_own_launch(call, segs):
    src, tgt, conn = CALLS[call](SEGS[segs])
    ops = [("create", 0, N)] + [("connect", src, tgt, conn, y, -1) for y in (SYN, SYN_C)]
    compare_all({"name": f"{call} over {segs}", "P": 1, "seed": 12, "dt": 0.1, "ops": ops}, 0)


def _batches(calls, batch):
    """The calls submitted in batches against connecting them one by one: the same arrays."""
    import paper_2512_09502_amd as snnc
    one = snnc.Network(1, 0, 12, 0.1)
    many = snnc.Network(1, 0, 12, 0.1)
    for net in (one, many):
        net.create(0, N)
    many.set_resident_budget(1 << 30)
    for src, tgt, conn, syn in calls:
        one.connect(src, tgt, conn, syn)
    for lo in range(0, len(calls), batch):
        st = many.submit_many(calls[lo:lo + batch], -1)
        assert all(s == 0 for s, _ in st)
        many.flush()
    for name in GEN_ARRAYS + ["call_off"]:
        got, ref = many.array(name), one.array(name)
        compare(name, got, ref, f"batches of {batch}")
        assert name != "gen_weight" or (got == ref).all()
    for net in (one, many):
        net.close()


BIG = (ALL, ALL, _conn("fixed_indegree", n=90), SYN)    # 5.4e5 connections: with it a batch uses both launches


@pytest.mark.parametrize("batch,big", [(1, False), (7, False), (64, False), (64, True)])
def test_batches_of_mixed_calls(batch, big):
    calls = [BIG] * big
    for k, (name, call) in enumerate(CALLS.items()):
        for j, segs in enumerate(SEGS.values()):
            src, tgt, conn = call(segs)
            calls.append((src, tgt, conn, SYN if (k + j) % 3 else SYN_C))
    log(f"mixed calls in batches of {batch}, large one {big}")
    _batches(calls, batch)


@pytest.mark.parametrize("n", [1, 2, 255, 1023, 1024, 1025])
@pytest.mark.parametrize("big", [False, True])
def test_batches_of_small_calls(n, big):
    """Requests on both sides of the line between the two launches, alone and beside a large one."""
    calls = [(ALL, [(0, 11 * k, 1)], _conn("fixed_indegree", n=n), SYN) for k in range(70)]
    calls += [(ALL, ALL, _conn("fixed_total_number", n=n), SYN_C), (ALL, [(0, 7, 2)], _conn("fixed_outdegree", n=3), SYN)]
    if big:
        calls.insert(30, BIG)
    log(f"small calls of {n}, large one {big}")
    _batches(calls, 40)


def _gen_us(make, reps=5):
    """Mean time of the generation launches of a repetition of make(net)."""
    import paper_2512_09502_amd as snnc
    net = snnc.Network(1, 0, 12, 0.1)
    net.create(0, 40000)
    net.set_resident_budget(1 << 30)
    make(net)
    net.sync()
    net.set_timing(1)
    for _ in range(reps):
        make(net)
    net.sync()
    us = sum(ms for k, (_, ms) in net.kernel_times().items() if k.startswith("gen")) / reps * 1e3
    net.close()
    return us


@pytest.mark.parametrize("case", ["one_to_one", "indegree", "floyd", "batch"])
def test_cost_of_short_runs(case):
    """Generation does a tile's draws once however many runs or calls it meets: at most eight times the launches of the
    same connections in one run, and 100 us (taken run by run it was 20 to 100 times)."""
    whole, parts = [(0, 0, 2000)], [(0, 2 * k, 1) for k in range(2000)]
    other = [(0, 20000, 2000)]
    if case == "batch":
        conn = _conn("fixed_indegree", n=1)
        few, many = [[(other, s, conn, SYN) for s in t] for t in ([whole], [[p] for p in parts])]

        def make(calls):
            return lambda net: (net.submit_many(calls, -1), net.flush())
        t_few, t_many = _gen_us(make(few)), _gen_us(make(many))
    else:
        conn = {"one_to_one": _conn("one_to_one"), "indegree": _conn("fixed_indegree", n=2),
                "floyd": _conn("fixed_indegree", n=2, multapses=False)}[case]
        t_few, t_many = [_gen_us(lambda net, t=t: net.connect(other, t, conn, SYN)) for t in (whole, parts)]
    log(f"{case}: one run {t_few:.1f} us, 2,000 runs {t_many:.1f} us")
    assert t_many <= 8 * t_few + 100
