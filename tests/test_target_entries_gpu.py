"""Prepare where the targets lie in many segments: parity on both sides of the
line (128 segments and one per 8,192 connections) up to which keys are written
in target order, and no time lost over it on the host."""
import time

import pytest

from gpu_util import compare_all, log
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu

SYN = {"weight": W.W_E, "delay": {"kind": "normal", "mean": 1.5, "sd": 0.75, "lo": 0.1}}


def _in(K):
    return {"rule": "fixed_indegree", "n": K, "autapses": True, "multapses": True}


@pytest.mark.parametrize("segs", [127, 128, 129, 130, 200])
@pytest.mark.parametrize("K", [16, 130])
def test_segments_of_one_call(segs, K):
    tgt = [(0, 1 + 3 * k, 2) for k in range(segs)]
    script = {"name": f"{segs} segments, K={K}", "P": 1, "seed": 4, "dt": 0.1,
              "ops": [("create", 0, 700), ("connect", [(0, 0, 600)], tgt, _in(K), SYN, -1)]}
    assert compare_all(script, 0) == 2 * segs * K


@pytest.mark.parametrize("calls", [10, 20, 40])
def test_overlapping_calls(calls):
    """Each call's targets overlap those of the calls around it: entries grow with the square of the calls."""
    ops = [("create", 0, 400), ("create", 1, 300)]
    ops += [("connect", [(k % 2, 10, 200)], [(0, 5 * k, 150)], _in(20), SYN, -1) for k in range(calls)]
    for host in (0, 1):
        compare_all({"name": f"{calls} calls", "P": 2, "seed": 4, "dt": 0.1, "ops": ops}, host)


def test_time_of_many_segments():
    """16,384 targets in segments of one take no more than twice as long as in one segment, and 100 us."""
    import paper_2512_09502_amd as snnc

    def seconds(tgt):
        best = 1e9
        for _ in range(7):
            net = snnc.Network(1, 0, 1, 0.1)
            net.create(0, 65536)
            net.connect([(0, 0, 65536)], tgt, _in(20), SYN)
            net.sync()
            t0 = time.perf_counter()
            net.prepare()
            best = min(best, time.perf_counter() - t0)
            net.close()
        return best

    one, many = seconds([(0, 0, 16384)]), seconds([(0, 4 * k, 1) for k in range(16384)])
    log(f"prepare: one segment {one * 1e6:.0f} us, 16,384 segments {many * 1e6:.0f} us")
    assert many <= 2 * one + 100e-6
