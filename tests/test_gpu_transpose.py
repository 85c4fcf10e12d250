"""The incidence transpose at the edges of its tiles, ranges and row classes.

Every row is compared with a stable sort of the (pin, net) pairs (exactly:
whole numbers), through both paths: vertex ranges finished in LDS, and the
radix sort that takes over where a range does not fit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2010_10272_amd import hgref
    return hgref


def rows_of_degrees(n, degrees, m, seed):
    """Net CSR in which vertex v has degrees[v] pins (the rest about 3), every
    net non-empty, no vertex twice in a net."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(1, 6, n)
    deg[:len(degrees)] = degrees
    nets = np.concatenate([rng.choice(m, d, replace=False) for d in deg])
    pins = np.repeat(np.arange(n), deg)
    empty = np.setdiff1d(np.arange(m), nets)
    nets, pins = np.concatenate([nets, empty]), np.concatenate([pins, rng.integers(0, n, empty.size)])
    order = np.lexsort((rng.random(nets.size), nets))        # pins of a net in any order
    eptr = np.concatenate(([0], np.cumsum(np.bincount(nets, minlength=m))))
    return eptr.astype(np.int64), pins[order].astype(np.int32)


def with_pins(P, n, seed):
    """P pins in two-pin nets (the last has one when P is odd)."""
    rng = np.random.default_rng(seed)
    a = rng.integers(0, n, (P + 1) // 2)
    pins = np.stack([a, (a + 1 + rng.integers(0, n - 1, a.size)) % n], 1).reshape(-1)[:P]
    eptr = np.minimum(np.arange(0, P + 2, 2), P)
    return eptr[:(P + 1) // 2 + 1].astype(np.int64), pins.astype(np.int32)


def bucket_of(pins_in_first, n, seed):
    """Two-pin nets whose first 512 vertices hold so many pins, the other vertices
    two each."""
    rng = np.random.default_rng(seed)
    a = np.arange(pins_in_first) % 512
    b = 512 + np.arange(pins_in_first) % (n - 512)
    more = 512 + rng.permutation(n - 512)[:(n - 512) // 2 * 2]
    pins = np.concatenate([np.stack([a, b], 1).ravel(), more])
    return np.arange(0, pins.size + 2, 2)[:pins.size // 2 + 1].astype(np.int64), pins.astype(np.int32)


def clustered(n, degrees, m, seed):
    """m nets, each with a pin of its own; vertex v in degrees[v] consecutive ones."""
    rng = np.random.default_rng(seed)
    nets, pins = [np.arange(m)], [rng.integers(len(degrees), n, m)]
    for v, d in enumerate(degrees):
        nets.append(rng.integers(0, m - d) + np.arange(d))
        pins.append(np.full(d, v))
    nets, pins = np.concatenate(nets), np.concatenate(pins)
    order = np.lexsort((rng.random(nets.size), nets))
    eptr = np.concatenate(([0], np.cumsum(np.bincount(nets, minlength=m))))
    return eptr.astype(np.int64), pins[order].astype(np.int32)


def hub_and(n, m, seed):
    """m nets of two pins and more, every one of them with vertex 0, in 12,000 nets."""
    m += 12_000
    rng = np.random.default_rng(seed)
    more = rng.integers(1, 4, m)
    pins = np.concatenate([np.concatenate(([0], 1 + rng.choice(n - 1, c, replace=False)))
                           for c in more])
    return np.concatenate(([0], np.cumsum(more + 1))).astype(np.int64), pins.astype(np.int32)


CASES = {
    # pins around one and two tiles of 8192, vertices around a bucket's width
    "tile-1": lambda: (700, *with_pins(8191, 700, 1)),
    "tile": lambda: (512, *with_pins(8192, 512, 2)),
    "tile+1": lambda: (513, *with_pins(8193, 513, 3)),
    "two-tiles": lambda: (70_001, *with_pins(2 * 8192 + 1, 70_001, 4)),
    "one-net": lambda: (5, np.array([0, 5], np.int64), np.array([4, 0, 3, 1, 2], np.int32)),
    "one-vertex": lambda: (1, np.arange(9, dtype=np.int64), np.zeros(8, np.int32)),
    # rows on both sides of every class: 16, 32, 512
    "row-classes": lambda: (3000, *rows_of_degrees(3000, [16, 17, 32, 33, 64, 65, 511, 512, 513,
                                                          1500], 2000, 5)),
    # rows on both sides of what a wavefront ranks, alone, many in a bucket, and more
    # of them than a bucket can hold of the next class
    "row-128": lambda: (3000, *rows_of_degrees(3000, [127, 128, 129, 130, 255, 256, 257], 900, 10)),
    "row-many-129": lambda: (2500, *rows_of_degrees(2500, [129] * 70, 4000, 11)),
    "row-many-600": lambda: (3000, *rows_of_degrees(3000, [600] * 15, 5000, 12)),
    "row-9000": lambda: (40_000, *rows_of_degrees(40_000, [9000], 12_000, 13)),
    # the same where the nets of a long row lie close together (radix passes in LDS)
    "row-clustered": lambda: (20_000, *clustered(20_000, [3000, 200, 129, 1200, 700], 80_000, 22)),
    "row-two-thirds": lambda: (300, *rows_of_degrees(300, [4000, 2, 4900], 5000, 14)),
    # a bucket (512 vertices here) that the LDS rows just hold, and one pin more, which
    # leaves all pins to the radix sort
    "bucket-full": lambda: (150_000, *bucket_of(10_240, 150_000, 15)),
    "bucket-over": lambda: (150_000, *bucket_of(10_241, 150_000, 15)),
    # 1,024 vertices a bucket: every place of its tables
    "wide-buckets": lambda: (5_000_000, *with_pins(6_000_000, 5_000_000, 16)),
    # the radix sort's first pass finds the nets: whole tiles of 4,096 and 8,192 pins (from
    # 2^24 pins on) and one pin more, nets across tiles, single-pin nets, one net over
    # many tiles
    "radix-tiles": lambda: (1, np.arange(16_385, dtype=np.int64), np.zeros(16_384, np.int32)),
    "radix-tiles+1": lambda: (1, np.arange(16_386, dtype=np.int64), np.zeros(16_385, np.int32)),
    "radix-hub": lambda: (200, *hub_and(200, 8191, 17)),
    "radix-single-pins": lambda: (3, np.arange(40_001, dtype=np.int64),
                                  (np.arange(40_000) % 3).astype(np.int32)),
    "radix-one-net": lambda: (9_000_000, np.array([0, 4_000_001], np.int64),
                              np.random.default_rng(20).permutation(9_000_000)[:4_000_001]
                              .astype(np.int32)),
    "radix-long-tiles": lambda: (9_000_000, *with_pins((1 << 24) + 5, 9_000_000, 21)),
    # a vertex in 30,000 nets: no bucket holds it, the radix sort takes over
    "hub": lambda: (9000, *rows_of_degrees(9000, [30_000], 30_000, 6)),
    # long nets across tiles, and more than one coarse range of 64 buckets
    "wide": lambda: (200_003, *with_pins(900_001, 200_003, 7)),
    "long-nets": lambda: (20_000, np.arange(0, 60_001, 20_000, dtype=np.int64),
                          np.concatenate([np.random.default_rng(8 + i).permutation(20_000)
                                          for i in range(3)]).astype(np.int32)),
    # few pins for many vertices: most rows empty (radix sort)
    "sparse-rows": lambda: (3_000_000, *with_pins(5000, 3_000_000, 9)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_incidence_rows(H, name):
    n, eptr, pins = CASES[name]()
    g = H.hg_load_csr(n, eptr, pins, k_max=2)
    net = np.repeat(np.arange(eptr.size - 1), np.diff(eptr))
    order = np.argsort(pins, kind="stable")
    vptr = np.concatenate(([0], np.cumsum(np.bincount(pins, minlength=n))))
    assert np.array_equal(g.vptr.cpu().numpy(), vptr)
    assert np.array_equal(g.vnets.cpu().numpy(), net[order])
    assert H.hg_get_info(g)["max_degree"] == int(np.diff(vptr).max())


@pytest.mark.parametrize("degree", [2, 16, 20, 32, 40, 600])
def test_repeated_pin_rejected(H, degree):
    """A vertex twice in one net, its row in every row class."""
    eptr, pins = rows_of_degrees(2000, [degree - 1], 1500, degree)
    e = int(np.searchsorted(eptr, np.nonzero(pins == 0)[0][0], side="right") - 1)
    pins = np.insert(pins, eptr[e], 0)
    eptr = eptr + (np.arange(eptr.size) > e)
    with pytest.raises(H.HgError, match="twice"):
        H.hg_load_csr(2000, eptr, pins, k_max=2)


@pytest.mark.parametrize("degree", [128, 129, 200, 1400])
@pytest.mark.parametrize("others", [0, 40])
def test_repeated_pin_rejected_in_long_rows(H, degree, others):
    """The same in the rows that a workgroup sorts together."""
    eptr, pins = rows_of_degrees(2000, [degree - 1] + [150] * others, 1500, degree)
    e = int(np.searchsorted(eptr, np.nonzero(pins == 0)[0][0], side="right") - 1)
    pins = np.insert(pins, eptr[e], 0)
    eptr = eptr + (np.arange(eptr.size) > e)
    with pytest.raises(H.HgError, match="twice"):
        H.hg_load_csr(2000, eptr, pins, k_max=2)


# Two fifths more than the load without such rows: what sorting a bucket's pins in one
# workgroup may add to a load that all workgroups share.  (Row after row, or a
# wavefront a row, they took one and a half to four times the load.)
@pytest.mark.parametrize("degrees", [[200] * 40, [450] * 18, [600] * 15],
                         ids=["40x200", "18x450", "15x600"])
def test_time_of_long_rows(H, degrees):
    import torch
    n, m, ms = 100_000, 100_000, []
    for degs in (degrees, []):
        eptr, pins = rows_of_degrees(n, degs, m, 7)
        ep, pn = torch.from_numpy(eptr).cuda(), torch.from_numpy(pins).cuda()
        out = (torch.empty(n + 1, dtype=torch.int64, device="cuda"),
               torch.empty(pins.size, dtype=torch.int32, device="cuda"),
               torch.empty(H.hg_workspace_size(n, m, pins.size, 2), dtype=torch.uint8,
                           device="cuda"))
        best = float("inf")
        for _ in range(15):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            H.hg_load_csr(n, ep, pn, k_max=2, out=out)
            ev[1].record()
            ev[1].synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]))
        ms.append(best)
    assert ms[0] < 1.4 * ms[1], ms
