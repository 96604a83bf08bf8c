"""GPU parity of the image numbering where source prefixes need more than 32
bits (remote hosts of about 2^31 neurons each, of which a call names a few):
spans at, one below and one above 2^32, up to the 48 bits of a key; every tile
shape, with earlier tiles counted instead of waited for, every sort algorithm,
keys in target order and not."""
import pytest

from gpu_util import compare_all
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu

BIG = 2**31 - 1
SYN = {"weight": W.W_E, "delay": {"kind": "normal", "mean": 1.5, "sd": 0.75, "lo": 0.1}}


def _conn(rule, n):
    return {"rule": rule, "n": n, "autapses": True, "multapses": True}


def _script(name, M, remote, target_order=True, K=40, **kw):
    """M neurons here, remote[h - 1] on host h; sources at both ends of every host's ids."""
    hosts = range(1, len(remote) + 1)
    last = [(h, n - 30, 30) for h, n in zip(hosts, remote)]
    first = [(h, 0, 20 + h) for h in reversed(hosts)]
    calls = [([(0, 0, M)], [(0, 0, M)], _conn("fixed_indegree", K)), (last, [(0, 5, M - 9)], _conn("fixed_indegree", 2 * K)),
             (first + last[:1], [(0, 0, M // 2)], _conn("fixed_indegree", 3 * K + 1))]
    if not target_order:
        calls += [(last[:2], [(0, 0, M)], _conn("fixed_outdegree", 7))]
    ops = [("create", 0, M)] + [("create", h, n) for h, n in zip(hosts, remote)]
    ops += [("connect", s, t, c, SYN, -1) for s, t, c in calls]
    return {"name": name, "P": 1 + len(remote), "seed": 8, "dt": 0.1, "ops": ops, **kw}


@pytest.mark.parametrize("target_order", [True, False])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_spans_around_32_bits(over, target_order):
    """Prefixes 0 .. M + G - 1 with M + G = 2^32 + over, the last neuron of the last host among the sources."""
    M = 60
    rest = 2**32 + over - 2 * M - BIG
    compare_all(_script(f"span 2^32 {over:+d}", M, [BIG, rest], target_order), 0)


@pytest.mark.parametrize("target_order", [True, False])
@pytest.mark.parametrize("M,hosts", [(60, 3), (300, 9), (4096, 31)])
def test_wide_spans(M, hosts, target_order):
    compare_all(_script(f"{hosts} hosts of 2^31 - 1", M, [BIG] * hosts, target_order), 0)


@pytest.mark.parametrize("spins", [0, 4096])
@pytest.mark.parametrize("variant", range(12))
def test_tile_shapes(variant, spins):
    compare_all(_script(f"shape {variant}", 700, [BIG] * 3, K=30, tune={"number_variant": variant, "lookback_spins": spins}), 0)


@pytest.mark.parametrize("tune", [{"sort_variant": v} for v in (1, 6, 12)] + [{"sort_mode": 1}, {"digit_bits": 8}, {"digit_bits": 9}])
def test_sort_settings(tune):
    compare_all(_script(str(tune), 500, [BIG] * 3, tune=tune), 0)


def _among_wide_hosts(n1):
    sizes = [BIG, n1, 5000, BIG, BIG]
    ops = [("create", h, n) for h, n in enumerate(sizes)]
    ops += [("connect", [(0, BIG - 50, 50), (3, 7, 40)], [(1, 0, 300)], _conn("fixed_indegree", 30), SYN, -1),
            ("connect", [(1, n1 - 100, 100)], [(2, 11, 200), (1, n1 - 1000, 1000)], _conn("fixed_indegree", 20), SYN, -1)]
    return {"name": f"{n1} neurons among wide hosts", "P": 5, "seed": 8, "dt": 0.1, "ops": ops}


@pytest.mark.parametrize("n1,pl", [(2**15, 1), (100_000, 2)])
def test_shares_of_smaller_hosts(n1, pl):
    """Two hosts of ordinary size among wide ones: sources and targets on both, the wide ones on either side."""
    compare_all(_among_wide_hosts(n1), pl)


def test_refused_beyond_48_bits():
    """33 bits of sources and 17 of targets."""
    import paper_2512_09502_amd as snnc
    with pytest.raises(snnc.SnncError) as e:
        snnc.run_script(_among_wide_hosts(100_000), 1)
    assert e.value.code == -5 and "48 key bits" in str(e.value)
