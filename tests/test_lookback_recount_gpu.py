"""GPU checks of the look-back of the radix and numbering passes at every tile
size that the library chooses by itself: sizes at the edges of the groups of
128 tiles that are dealt over the dies, and passes that take no earlier tile's
counts and so count every one themselves ("lookback_recount")."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILES = {8: 4096, 0: 8192, 12: 16384}      # sort_variant: pairs a tile
GROUP = 128


def _check(n, bits, variant, **tune):
    import torch
    import paper_2512_09502_amd as snnc
    torch.cuda.set_device(0)
    print(f"look-back n={n} bits={bits} variant={variant} {tune}", flush=True)
    net = snnc.Network(1, 0, 1, 0.1)
    net.tune("sort_variant", variant)
    for key, value in tune.items():
        net.tune(key, value)
    rng = np.random.default_rng(n + bits)
    keys = rng.integers(0, 2**40, size=n, dtype=np.int64)
    keys[: n // 3] &= ~np.int64(0xff << 16)               # tiles without most digits
    vals = np.arange(n, dtype=np.int32)
    for _ in range(2):                                    # the second call meets the first one's table
        k, v = net.sort_pairs(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda(), 16, 16 + bits)
        order = np.argsort((keys >> 16) & ((1 << bits) - 1), kind="stable")
        np.testing.assert_array_equal(v.cpu().numpy(), order.astype(np.int32))
        np.testing.assert_array_equal(k.cpu().numpy(), keys[order])
    net.close()


@pytest.mark.parametrize("variant", TILES)
@pytest.mark.parametrize("bits", [16, 18])                # two 8-bit or two 9-bit digits
@pytest.mark.parametrize("tiles,rest", [(1, 0), (2, 1), (5, 77), (9, -1)])
def test_every_tile_counted(variant, bits, tiles, rest):
    _check(tiles * TILES[variant] + rest, bits, variant, lookback_spins=0, lookback_recount=1)


@pytest.mark.parametrize("spins", [0, 4096])
@pytest.mark.parametrize("variant", TILES)
@pytest.mark.parametrize("bits", [16, 18])
@pytest.mark.parametrize("groups,rest", [(1, -1), (1, 0), (1, 1), (2, 4097)])
def test_tile_groups(variant, bits, spins, groups, rest):
    _check(groups * GROUP * TILES[variant] + rest, bits, variant, lookback_spins=spins)


@pytest.mark.parametrize("variant", [0, 3, 4, 5, 6, 7, 8, 10, 11])
@pytest.mark.parametrize("wide", [False, True])
def test_numbering_counts_every_tile(variant, wide):
    from gpu_util import compare_all
    from paper_2512_09502_amd import workloads as W
    tune = {"lookback_spins": 0, "lookback_recount": 1, "number_variant": variant}
    if wide:
        big, y = 2**31 - 1, {"weight": W.W_E, "delay": {"kind": "const", "mean": 0.3}}
        conn = {"rule": "fixed_indegree", "n": 90, "autapses": True, "multapses": True}
        ops = [("create", 0, 500)] + [("create", h, big) for h in (1, 2, 3)]
        ops += [("connect", [(h, big - 300, 300)], [(0, 0, 500)], conn, y, -1) for h in (1, 2, 3)]
        compare_all({"name": f"wide {variant}", "P": 4, "seed": 2, "dt": 0.1, "ops": ops, "tune": tune}, 0)
    else:
        s = W.balanced_collective(P=7, n_e=400, n_i=100, k_e=180, k_i=45)
        s["tune"] = tune
        compare_all(s, 3)


def test_setting_range():
    import paper_2512_09502_amd as snnc
    net = snnc.Network(1, 0, 1, 0.1)
    for bad in (-1, 2):
        with pytest.raises(snnc.SnncError):
            net.tune("lookback_recount", bad)
    net.close()
