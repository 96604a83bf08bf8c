"""GPU checks of the radix pass's tile order and look-back: sizes at the edges
of the 64-tile groups that are dealt over the dies, and look-backs that count
earlier tiles themselves instead of waiting (lookback_spins down to 0)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.mark.parametrize("spins", [0, 2, 4096])
@pytest.mark.parametrize("bits", [16, 18])                # two 8-bit or two 9-bit digits
@pytest.mark.parametrize("n", [TILE, 2 * TILE + 1, 64 * TILE - 1, 64 * TILE, 64 * TILE + 1, 130 * TILE + 77])
def test_tile_order(spins, bits, n):
    import torch
    import paper_2512_09502_amd as snnc
    torch.cuda.set_device(0)
    net = snnc.Network(1, 0, 1, 0.1)
    net.tune("lookback_spins", spins)
    rng = np.random.default_rng(n + bits)
    keys = rng.integers(0, 2**40, size=n, dtype=np.int64)
    keys[: n // 3] &= ~np.int64(0xff << 16)               # tiles without most digits
    vals = np.arange(n, dtype=np.int32)
    k, v = net.sort_pairs(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda(), 16, 16 + bits)
    order = np.argsort((keys >> 16) & ((1 << bits) - 1), kind="stable")
    np.testing.assert_array_equal(v.cpu().numpy(), order.astype(np.int32))
    np.testing.assert_array_equal(k.cpu().numpy(), keys[order])
    net.close()


@pytest.mark.parametrize("spins", [0, 1, 4096])
@pytest.mark.parametrize("variant", [7, 10])              # 256 x 6 and 1024 x 10 items a tile
def test_numbering_counts_missing_tiles(spins, variant):
    from gpu_util import compare_all
    from paper_2512_09502_amd import workloads as W
    s = W.balanced_collective(P=7, n_e=400, n_i=100, k_e=180, k_i=45)
    s["tune"] = {"lookback_spins": spins, "number_variant": variant}
    compare_all(s, 3)


def test_spin_limit_range():
    import paper_2512_09502_amd as snnc
    net = snnc.Network(1, 0, 1, 0.1)
    for bad in (-1, (1 << 22) + 1):
        with pytest.raises(snnc.SnncError):
            net.tune("lookback_spins", bad)
    net.close()
