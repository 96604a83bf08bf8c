"""Errors of the spike exchange leave the caller's arrays alone: an invalid
spike id writes no packet, an entry outside its map (per-entry outputs are
written) no event, a small capacity neither; the next valid call is not
affected.  Sizes on both sides of the one-workgroup packets and of a delivery
block, the invalid one first, last and in between."""
import ctypes

import numpy as np
import pytest

import oracle
from gpu_util import log
from paper_2512_09502_amd import workloads as W

pytestmark = pytest.mark.gpu


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=np.uint32)).view(np.int32)).cuda()


def _full(n, dtype):
    import torch
    t = torch.empty(n, dtype=dtype, device="cuda")
    t.view(torch.uint8).fill_(0x5A)
    return t


def _untouched(t):
    import torch
    return bool((t.view(torch.uint8) == 0x5A).all())


@pytest.fixture(scope="module")
def nets():
    import torch
    import paper_2512_09502_amd as snnc
    torch.cuda.set_device(0)
    p2p = W.multiarea_p2p(P=6, n_e=1600, n_i=400, k_e=40, k_i=10, k_remote_max=12, seed=21)
    coll = W.balanced_collective(P=12, n_e=1600, n_i=400, k_e=90, k_i=22)
    out = {k: (snnc.run_script(s, 1), oracle.run_script(s, 1)) for k, s in ((0, p2p), (1, coll))}
    yield out
    for g, _ in out.values():
        g.close()


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [1, 50, 1025, 3000])
def test_packets(nets, kind, n):
    import torch
    import paper_2512_09502_amd as snnc
    gnet, onet = nets[kind]
    M, n_dest = onet.neurons(1), (6 if kind == 0 else onet.array("groups").size)
    rng = np.random.default_rng(n)
    good = rng.integers(0, M, size=n)
    ref = onet.spike_packets(kind, good, None)
    total = int(ref["off"][-1])
    cap = max(1, total)
    for at, cap_here in [(0, cap), (n // 2, cap), (n - 1, cap), (n - 1, 0), (None, total - 1)]:
        if cap_here < 0:
            continue
        spikes = good.copy()
        if at is not None:
            spikes[at] = M + at
        log(f"packets kind={kind} n={n} at={at} cap={cap_here}")
        off, pos, mult = _full(n_dest + 1, torch.int64), _full(cap, torch.int32), _full(cap, torch.int32)
        n_out, dev = ctypes.c_uint64(77), _dev(spikes)
        st = snnc.lib().snnc_spike_packets(gnet._h, kind, _ptr(dev), None, n, _ptr(off), _ptr(pos), _ptr(mult),
                                           cap_here, ctypes.byref(n_out))
        assert st == -1 and n_out.value == (77 if at is not None else total)
        assert _untouched(off) and _untouched(pos) and _untouched(mult)
        got = gnet.spike_packets(kind, _dev(good))
        np.testing.assert_array_equal(got["off"].cpu().numpy().view(np.uint64), ref["off"])
        np.testing.assert_array_equal(got["pos"].cpu().numpy().view(np.uint32), ref["pos"])


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [1, 37, 1024, 1025, 5000])
def test_delivery(nets, kind, n):
    import torch
    import paper_2512_09502_amd as snnc
    gnet, onet = nets[kind]
    size = np.diff(onet.array("r_off" if kind == 0 else "h_off").astype(np.int64))[: 6 if kind == 0 else 12]
    rng = np.random.default_rng(n + kind)
    host = rng.choice(np.flatnonzero((size > 0) & (np.arange(size.size) != 1)), size=n)
    pos = rng.integers(0, size[host])
    grp = _dev(np.zeros(n)) if kind == 1 else None
    ref = onet.deliver(kind, host, pos, None, np.zeros(n) if kind == 1 else None)
    cap = max(1, ref["tgt"].size)
    d_host = _dev(host)
    for at, cap_here in [(0, cap), (n // 2, cap), (n - 1, cap), (n - 1, 0), (None, ref["tgt"].size - 1)]:
        if cap_here < 0:
            continue
        log(f"delivery kind={kind} n={n} at={at} cap={cap_here}")
        p = pos.copy()
        if at is not None:
            p[at] = size[host[at]] + at                     # past its map
        d_pos = _dev(p)
        image, rb, re = _full(n, torch.int32), _full(n, torch.int64), _full(n, torch.int64)
        et, ed, ew = _full(cap, torch.int32), _full(cap, torch.int16), _full(cap, torch.float32)
        n_ev = ctypes.c_uint64(77)
        st = snnc.lib().snnc_deliver(gnet._h, kind, _ptr(grp), _ptr(d_host), _ptr(d_pos), None, n, _ptr(image),
                                     _ptr(rb), _ptr(re), _ptr(et), _ptr(ed), _ptr(ew), cap_here, ctypes.byref(n_ev))
        assert st == -1 and n_ev.value == (77 if at is not None else ref["tgt"].size)
        assert _untouched(et) and _untouched(ed) and _untouched(ew)
        keep = np.arange(n) != (n if at is None else at)      # the other entries' outputs are written
        np.testing.assert_array_equal(image.cpu().numpy()[keep], ref["image"][keep])
        np.testing.assert_array_equal(rb.cpu().numpy().view(np.uint64)[keep], ref["row_begin"][keep])
        np.testing.assert_array_equal(re.cpu().numpy().view(np.uint64)[keep], ref["row_end"][keep])
        got = gnet.deliver(kind, d_host, _dev(pos), None, grp)
        np.testing.assert_array_equal(got["tgt"].cpu().numpy(), ref["tgt"])
        np.testing.assert_array_equal(got["weight"].cpu().numpy().view(np.uint32), ref["weight"].view(np.uint32))
