"""Sorts of no pairs: accepted by both entry points, nothing written, the
result in the caller's first arrays; at every tile shape, pass algorithm and
digit width."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [None, 0, 1, 8, 12])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("lo,hi", [(0, 0), (16, 24), (16, 34), (0, 64)])
def test_no_pairs(variant, mode, lo, hi):
    import torch
    import paper_2512_09502_amd as snnc
    torch.cuda.set_device(0)
    net = snnc.Network(1, 0, 1, 0.1)
    if variant is not None:
        net.tune("sort_variant", variant)
        net.tune("sort_mode", mode)
    k, v = (torch.empty(0, dtype=t, device="cuda") for t in (torch.int64, torch.int32))
    for got in (net.sort_pairs(k, v, lo, hi),
                net.sort_pairs_noalloc(k, v, torch.empty_like(k), torch.empty_like(v), lo, hi)):
        assert got[0] is k and got[1] is v
    keys = torch.tensor([5 << 16, 1 << 16, 3 << 16], device="cuda")      # the context still sorts
    sk, sv = net.sort_pairs(keys, torch.arange(3, dtype=torch.int32, device="cuda"), 16, 24)
    assert sk.tolist() == [1 << 16, 3 << 16, 5 << 16] and sv.tolist() == [1, 2, 0]
    net.close()
