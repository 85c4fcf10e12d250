"""Contraction at the edges of its units: nets around four LDS places, around the
longest that a wavefront takes (128 pins) and around what fits its LDS, net counts
around a wavefront and around the widths of the sort key; clusterings with few and
many duplicates.  Exactly equal to the oracle."""
import numpy as np
import pytest

import synth

from .test_gpu_contract import H, _check  # noqa: F401
from .test_gpu_counts import nets_of

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 4, 5, 7, 8, 9, 127, 128, 129, 130, 64, 1, 1, 200, 63, 65]


@pytest.mark.parametrize("m,n,sizes", [
    (1, 5, [4]), (1, 300, [129]), (63, 400, SIZES), (64, 400, SIZES), (65, 400, SIZES),
    (257, 400, [128]),                      # six nets fill a wavefront's places
    (130, 400, [129]),                      # long nets only: more than one list of 64
    (4096, 500, [2, 3]), (4097, 500, [2, 3]), ((1 << 20) + 1, 3000, [2])])
def test_edges(H, m, n, sizes):
    lens = [sizes[i % len(sizes)] for i in range(m)]
    if m < 10000:
        eptr, pins = nets_of(lens, n, m)
    else:
        eptr = 2 * np.arange(m + 1, dtype=np.int64)
        a = np.random.default_rng(m).integers(0, n - 1, m)
        pins = np.stack([a, a + 1], 1).ravel().astype(np.int32)
    w = np.random.default_rng(n).integers(1, 9, m).astype(np.int32)
    inst = synth.Instance("edges", n, eptr, pins, None, w, np.zeros(n, np.int32), 2, 0.03, 1)
    g = H.hg_load_csr(n, eptr, pins, None, w, k_max=2)
    rng = np.random.default_rng(m + n)
    for name, cl in (("alone", np.arange(n)), ("pairs", np.arange(n) // 2 * 2),
                     ("anywhere", rng.integers(0, n, n)), ("few", rng.integers(0, 5, n))):
        _check(H, g, inst, cl.astype(np.int32), (m, name))


@pytest.mark.parametrize("m,sizes", [
    (1, [2048]), (1, [2049]), (3, [2047, 2048, 2049]), (70, [2, 3000, 5]),
    (90, [100]), (300, [40]), (8192, [16, 17]), (500, [127, 1, 129, 300])])
def test_edges_of_long_nets_and_units(H, m, sizes):
    """Nets around the longest that a wavefront writes out (2048 pins), and net counts
    and sizes for which a wavefront takes fewer than 64 nets."""
    n = 4096
    lens = [sizes[i % len(sizes)] for i in range(m)]
    rng = np.random.default_rng(m)
    step = 1 + 2 * rng.integers(0, 3, m)                 # odd, n a power of two: distinct pins
    start = rng.integers(0, n, m)
    pins = np.concatenate([(start[i] + np.arange(s) * step[i] % n) % n
                           for i, s in enumerate(lens)]).astype(np.int32)
    eptr = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
    inst = synth.Instance("long", n, eptr, pins, None, None, np.zeros(n, np.int32), 2, 0.03, 1)
    g = H.hg_load_csr(n, eptr, pins, None, None, k_max=2)
    for name, cl in (("alone", np.arange(n)), ("pairs", np.arange(n) // 2 * 2),
                     ("few", rng.integers(0, 5, n))):
        _check(H, g, inst, cl.astype(np.int32), (m, name))


# Half as much again as the same pins in nets of ten, which have ten times the nets to
# sort, compare and number.  (With 64 nets a wavefront whatever their length they took
# two to three times as long.)
@pytest.mark.parametrize("size,m", [(128, 10_000), (100, 30_000)])
def test_time_of_longer_nets(H, size, m):
    import torch
    n, ms = 100_000, []
    for s, count in ((size, m), (10, m * size // 10)):
        rng = np.random.default_rng(s)
        pins = ((rng.integers(0, n, count)[:, None] + 331 * np.arange(s)[None, :]) % n)
        eptr = s * np.arange(count + 1, dtype=np.int64)
        g = H.hg_load_csr(n, eptr, pins.astype(np.int32).ravel(), k_max=2)
        out, ws = H.Coarse(g), H.contract_workspace(g)
        cl = (torch.arange(n, device="cuda", dtype=torch.int32) // 2 * 2)
        best = float("inf")
        for _ in range(8):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            H.hg_contract(g, cl, out, ws)
            ev[1].record()
            ev[1].synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]))
        ms.append(best)
    assert ms[0] < 1.5 * ms[1], ms


@pytest.mark.parametrize("m,sizes", [(1, [129]), (5, [130, 200]), (257, [129]),
                                     (4099, [129, 3, 140]), (8200, [131])])
def test_edges_of_listed_nets(H, m, sizes):
    """Long nets only, or nearly so: few of them a wavefront, listed by workgroups."""
    test_edges_of_long_nets_and_units(H, m, sizes)


def test_time_of_listed_nets(H):
    """10,000 nets of 256 pins, a workgroup each, in half as much again as nets of 128:
    twice the pins, in a call half of which is launches.  (Listed by an atomic per
    wavefront of four nets they took 1.7 times as long.)"""
    import torch
    n, m, ms = 100_000, 10_000, []
    for size in (256, 128):
        rng = np.random.default_rng(size)
        pins = (rng.integers(0, n, m)[:, None] + 331 * np.arange(size)[None, :]) % n
        g = H.hg_load_csr(n, size * np.arange(m + 1, dtype=np.int64),
                          pins.astype(np.int32).ravel(), k_max=2)
        out, ws = H.Coarse(g), H.contract_workspace(g)
        cl = torch.arange(n, device="cuda", dtype=torch.int32) // 2 * 2
        best = float("inf")
        for _ in range(8):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            H.hg_contract(g, cl, out, ws)
            ev[1].record()
            ev[1].synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]))
        ms.append(best)
    assert ms[0] < 1.5 * ms[1], ms
