"""Nets of more than 255 pins (32-bit counters) and of more than 2048 (a workgroup
each): exact values at the edges of both, through every call that counts pins, and
no more time than the pins themselves take."""
import numpy as np
import pytest

import synth

from .test_gpu_counts import H, check, nets_of  # noqa: F401
from .test_gpu_finalize import _check_round

pytestmark = pytest.mark.gpu

EDGES = [254, 255, 256, 257, 511, 1024, 2047, 2048, 2049, 4095, 4096, 4097, 9000, 12000]
SHORT = [1 + i % 9 for i in range(500)]


def _case(k, n=12000):
    """Long nets alone in a wavefront's nets, many together, and among short ones."""
    sizes = EDGES + SHORT + [300] * 70 + [2, 3000, 2, 2500] + [1] * 64 + [2048, 2049]
    eptr, pins = nets_of(sizes, n, k)
    part = np.random.default_rng(k).integers(0, k, n).astype(np.int32)
    part[:n // 3] = k - 1                               # long runs of one block
    w = None if k % 2 == 0 else np.random.default_rng(k).integers(1, 5, len(sizes)).astype(np.int32)
    return n, eptr, pins, part, w


KS = [2, 3, 4, 8, 16, 17, 33, 64, 65, 128, 129, 256]


@pytest.mark.parametrize("k", KS)
def test_counts(H, k):
    n, eptr, pins, part, w = _case(k)
    _, st, km1 = check(H, eptr, pins, n, k, part, w)
    assert int(st.km1.item()) == km1


@pytest.mark.parametrize("m,size", [(1, 300), (3, 256), (65, 257), (64, 2048), (64, 2049), (2, 70000)])
@pytest.mark.parametrize("k", [2, 100])
def test_counts_of_equal_nets(H, k, m, size):
    n = size + 1000
    eptr, pins = nets_of([size] * m, n, m)
    part = np.random.default_rng(size).integers(0, k, n).astype(np.int32)
    check(H, eptr, pins, n, k, part)


@pytest.mark.parametrize("m,size", [(4096, 256), (4097, 64), (5000, 65), (4100, 300)])
@pytest.mark.parametrize("k", [2, 17, 64])
def test_counts_by_lane_groups(H, k, m, size):
    """Sizes that the pin counts hand to eight lanes a net, with a few other nets
    (a single pin, longer than a workgroup's share) among them."""
    n = 3000
    rng = np.random.default_rng(size)
    sizes = [size] * m
    sizes[7], sizes[8], sizes[-1] = 1, 2049, 2500
    start = rng.integers(0, n, m)
    pins = np.concatenate([(start[i] + np.arange(s)) % n for i, s in enumerate(sizes)])
    eptr = np.concatenate(([0], np.cumsum(sizes))).astype(np.int64)
    part = rng.integers(0, k, n).astype(np.int32)
    w = None if k % 2 == 0 else rng.integers(1, 5, m).astype(np.int32)
    _, st, km1 = check(H, eptr, pins.astype(np.int32), n, k, part, w)
    assert int(st.km1.item()) == km1
    part[3] = k                                       # counted nowhere
    g, _, _ = check(H, eptr, pins.astype(np.int32), n, k, part, w)
    with pytest.raises(H.HgError, match="partition id"):
        H.hg_sync_status(g)


@pytest.mark.parametrize("how", ["refine", "round", "noalloc", "cached", "exact"])
@pytest.mark.parametrize("k", KS)
def test_rounds(H, k, how):
    import torch
    n, eptr, pins, part, w = _case(k)
    g = H.hg_load_csr(n, eptr, pins, None, w, k_max=k)
    st = H.State(g, k, part)
    stats = torch.zeros(H.STATS_WORDS, dtype=torch.int64, device="cuda")
    H.hg_compute_pincounts(g, st)
    st.eligible.fill_(1)
    lmax, approved = H.hg_max_block_weight(g, k, 0.5), 0
    if how == "cached":
        cache = H.gain_cache(g, k)
        H.hg_gain_cache_init(g, k, st.part, st.netstate, cache)
    for _ in range(1 if how == "refine" else 2):
        before, km1 = st.part.cpu().numpy(), int(st.km1.item())
        if how == "refine":
            H.hg_refine(g, st, 0.5, 1, stats)
        elif how == "round":
            H.hg_lp_round(g, st, lmax, stats)
        elif how == "noalloc":
            H.hg_lp_round_noalloc(g, st, lmax, stats)
        elif how == "exact":
            H.hg_lp_round_exact(g, st, lmax, stats, H.moves_workspace(g, k))
        else:
            H.hg_lp_round_cached(g, st, lmax, stats, cache)
            want = H.gain_cache(g, k)
            H.hg_gain_cache_init(g, k, st.part, st.netstate, want)
            for a, b in zip(H.cache_views(g, k, cache), H.cache_views(g, k, want)):
                assert torch.equal(a, b)
        approved += _check_round(H, g, before, st, stats, eptr, pins, k, km1)
    assert approved > 0


@pytest.mark.parametrize("k", [4, 200])
def test_batch_and_server_equal_refine(H, k):
    import torch

    from .test_gpu_batch import _members, _snapshot
    insts = []
    for i in range(3):
        n, eptr, pins, part, w = _case(k, 12000 + i)
        insts.append(synth.Instance("long-%d" % i, n, eptr, pins, None, w, part, k, 0.1, 3))
    insts.append(synth.random_power_law(5, 3000, 3000, k, rounds=3, eps=0.1))
    for size in (64, 300):                              # eight lanes a net in a batch
        eptr, pins = nets_of([size] * 300, 3000, size)
        part = np.random.default_rng(size).integers(0, k, 3000).astype(np.int32)
        insts.append(synth.Instance("equal-%d" % size, 3000, eptr, pins, None, None, part, k, 0.1, 3))
    alone = []
    for mb, x in zip(_members(H, insts, 3), insts):
        H.hg_refine(mb.g, mb.st, x.eps, 3, mb.stats)
        alone.append(_snapshot(mb))
    members = _members(H, insts, 3)
    b = H.hg_batch_create(members)
    H.hg_batch_start(b)
    for r in range(3):
        H.hg_batch_round(b, r)
    torch.cuda.synchronize()
    for mb, want in zip(members, alone):
        for a, c in zip(_snapshot(mb), want):
            assert np.array_equal(a, c)
    for mb, x in zip(members, insts):
        mb.st.part.copy_(torch.from_numpy(x.part))
    H.hg_batch_refine(b, 3)
    torch.cuda.synchronize()
    for mb, want in zip(members, alone):
        for a, c in zip(_snapshot(mb), want):
            assert np.array_equal(a, c)
    b.free()
    srv = H.hg_server_create(1 << 30, table_bytes=8 << 20, max_active=4)
    ids = [H.hg_server_submit(srv, x.n, x.eptr, x.pins, x.part, x.k, 3, x.eps, vwgt=x.c, ewgt=x.w)
           for x in insts]
    assert H.hg_server_drain(srv, 60000.0) == 0
    for jid, want in zip(ids, alone):
        assert H.hg_server_info(srv, jid)["status"] == H.HG_OK
        assert np.array_equal(H.hg_server_result(srv, jid)[0].numpy(), want[0])
    srv.free()


def _best_ms(f):
    import torch
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    f()
    best = float("inf")
    for _ in range(7):
        ev[0].record()
        f()
        ev[1].record()
        ev[1].synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]))
    return best


# Twice the time of the same pins in nets of ten: the same gathers and stores, fewer
# rows.  (Nets that wait for one another take 4 to 100 times as long.)
@pytest.mark.parametrize("sizes", [[20_000] * 20, [1500] * 2000, [300_000], [3000] * 300],
                         ids=["20x20000", "2000x1500", "1x300000", "300x3000"])
@pytest.mark.parametrize("what", ["counts", "round"])
def test_time_of_long_nets(H, sizes, what):
    import torch
    n, k, P = 400_000, 8, sum(sizes)
    ms = []
    for lens in (sizes, [10] * (P // 10)):
        rng = np.random.default_rng(1)
        pins = np.concatenate([(rng.integers(0, n) + np.arange(s) * 7) % n for s in lens])
        eptr = np.concatenate(([0], np.cumsum(lens)))
        g = H.hg_load_csr(n, eptr.astype(np.int64), pins.astype(np.int32), k_max=k)
        st = H.State(g, k, np.arange(n, dtype=np.int32) % k)
        stats = torch.zeros(H.STATS_WORDS, dtype=torch.int64, device="cuda")
        part, lmax = st.part.clone(), H.hg_max_block_weight(g, k, 0.03)

        def counts():
            st.part.copy_(part)
            H.hg_compute_pincounts(g, st)

        def rounds():
            counts()
            st.eligible.fill_(1)
            H.hg_lp_round(g, st, lmax, stats)

        ms.append(_best_ms(counts if what == "counts" else rounds))
    # a tenth of a millisecond: steps of one net are a chain
    assert ms[0] < 2 * ms[1] + 0.1, ms


@pytest.mark.parametrize("k", [3, 64])
def test_counts_of_more_medium_nets_than_resident(H, k):
    """More workgroups of lane groups than reside at once, the last one with one net."""
    import torch
    n, m, size = 1 << 15, 4096 * 32 + 1, 64
    rng = np.random.default_rng(k)
    pins = (rng.integers(0, n, m)[:, None] + np.arange(size) * 3) % n
    part = rng.integers(0, k, n).astype(np.int32)
    g = H.hg_load_csr(n, np.arange(m + 1, dtype=np.int64) * size,
                      pins.reshape(-1).astype(np.int32), k_max=k)
    st = H.State(g, k, part)
    H.hg_compute_pincounts(g, st)
    phi = np.bincount((np.arange(m)[:, None] * k + part[pins]).reshape(-1), minlength=m * k)
    assert np.array_equal(st.phi.cpu().numpy().reshape(-1), phi)
    assert int(st.km1.item()) == int((phi.reshape(m, k) > 0).sum()) - m
    H.hg_sync_status(g)


# The same pins in nets of 300, which lane groups have counted all along, and a fifth.
# (With 64 nets a wavefront nets of 200 took half as long again, 160,000 in two turns a
# third.)
@pytest.mark.parametrize("size,m", [(200, 100_000), (200, 160_000)])
@pytest.mark.parametrize("k", [8, 64])
def test_time_of_medium_nets(H, size, m, k):
    n, ms = 1 << 17, []
    for s in (size, 300):
        nets = m * size // s
        rng = np.random.default_rng(1)
        pins = (rng.integers(0, n, nets)[:, None] + np.arange(s)) % n
        g = H.hg_load_csr(n, np.arange(nets + 1, dtype=np.int64) * s,
                          pins.reshape(-1).astype(np.int32), k_max=k)
        st = H.State(g, k, np.random.default_rng(2).integers(0, k, n).astype(np.int32))
        ms.append(_best_ms(lambda: [H.hg_compute_pincounts(g, st) for _ in range(10)]))
    assert ms[0] < 1.2 * ms[1], ms
