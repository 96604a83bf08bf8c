"""Device-memory budgets that hold a network with large sort tiles hold it with
any tile: where the look-back table of the chosen tiles does not fit, the sort
takes larger ones, and the table does not stay for the steps after it.  Same
arrays."""
import pytest

from gpu_util import PREP_ARRAYS, compare, log
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,size", [(7, (2000, 500, 800, 200)), (7, (4000, 1000, 200, 50)), (7, (3200, 800, 960, 240)),
                                    (7, (8000, 2000, 1600, 400)), (64, (1600, 400, 2400, 600))])
@pytest.mark.parametrize("gen_blocks", [0, 1])
def test_budget_of_large_tiles(P, size, gen_blocks):
    import paper_2512_09502_amd as snnc
    script = W.balanced_collective(P, *size)
    script["tune"] = {"gen_blocks": gen_blocks}
    large = snnc.run_script(dict(script, tune={"gen_blocks": gen_blocks, "sort_variant": 12}), 3, torch_allocator=False)
    peak = large.stats()["bytes_peak"]
    log(f"{large.count('src')} connections, budget {peak}")
    for tune in ({}, {"sort_variant": 8}, {"sort_variant": 0}):
        net = snnc.run_script(dict(script, tune={"gen_blocks": gen_blocks, **tune}), 3, torch_allocator=False,
                              budget_bytes=peak)
        for name in PREP_ARRAYS:
            compare(name, net.array(name), large.array(name), f"budget {peak} {tune}")
        net.close()
    large.close()


def test_refused_without_room_for_any_tile():
    import torch
    import paper_2512_09502_amd as snnc
    net = snnc.Network(1, 0, 1, 0.1, torch_allocator=False, budget_bytes=9 << 20)     # a slab and little more
    n = 40_000_000
    k, v = torch.zeros(n, dtype=torch.int64, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    with pytest.raises(snnc.SnncError) as e:
        net.sort_pairs(k, v, 16, 56)
    assert e.value.code == -3
    keys = torch.tensor([5 << 16, 1 << 16, 3 << 16], device="cuda")      # the context still sorts
    assert net.sort_pairs(keys, torch.arange(3, dtype=torch.int32, device="cuda"), 16, 24)[1].tolist() == [1, 2, 0]
    net.close()
