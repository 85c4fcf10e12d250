"""Pin counts at the edges of their units, counter widths and record widths,
against numpy (whole numbers, exactly)."""
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


def nets_of(sizes, n, seed):
    rng = np.random.default_rng(seed)
    pins = np.concatenate([np.sort(rng.choice(n, s, replace=False)) for s in sizes])
    return np.concatenate(([0], np.cumsum(sizes))).astype(np.int64), pins.astype(np.int32)


def expect(eptr, pins, part, k, w):
    m = eptr.size - 1
    net = np.repeat(np.arange(m), np.diff(eptr))
    ok = part[pins] < k
    phi = np.zeros((m, k), np.int64)
    np.add.at(phi, (net[ok], part[pins][ok]), 1)
    lam = (phi > 0).sum(1)
    return phi, lam, int(((lam - 1) * w).sum())


def check(H, eptr, pins, n, k, part, w=None, views=None):
    m = eptr.size - 1
    g = H.hg_load_csr(n, eptr, pins, None, w, k_max=k)
    st = H.State(g, k, part)
    H.hg_compute_pincounts(g, st)
    phi, lam, km1 = expect(eptr, pins, part, k, 1 if w is None else w)
    assert np.array_equal(st.phi.view(m, k).cpu().numpy(), phi)
    gw, glam, gset, gone = (x.cpu().numpy() for x in H.decode_netstate(st.netstate, m, k))
    assert np.array_equal(gw, np.ones(m) if w is None else w)
    assert np.array_equal(glam, lam)
    for words, want in ((gset, phi > 0), (gone, phi == 1)):
        bits = (words.astype(np.uint32)[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1
        assert np.array_equal(bits.reshape(m, -1)[:, :k].astype(bool), want)
    return g, st, km1


@pytest.mark.parametrize("k", [2, 3, 4, 5, 8, 16, 17, 32, 33, 64, 65, 128, 129, 256])
def test_widths(H, k):
    """Every record and counter width, nets on both sides of a byte counter's
    range (255 pins) among short ones."""
    n = 1500
    sizes = [1, 2, 255, 256, 257, 63, 64, 65, 1000, 3] + [1 + i % 7 for i in range(251)]
    eptr, pins = nets_of(sizes, n, k)
    part = np.random.default_rng(k).integers(0, k, n).astype(np.int32)
    part[:700] = k - 1                                  # one block fills long runs
    w = None if k % 2 else np.random.default_rng(k).integers(1, 5, len(sizes)).astype(np.int32)
    _, st, km1 = check(H, eptr, pins, n, k, part, w)
    assert int(st.km1.item()) == km1
    assert np.array_equal(st.block_w.cpu().numpy(), np.bincount(part, minlength=k))


@pytest.mark.parametrize("m", [1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 513])
@pytest.mark.parametrize("k", [16, 200])
def test_unit_edges(H, m, k):
    n = 777
    eptr, pins = nets_of([1 + (5 * i) % 11 for i in range(m)], n, m)
    part = np.random.default_rng(m).integers(0, k, n).astype(np.int32)
    check(H, eptr, pins, n, k, part)


@pytest.mark.parametrize("k,bad", [(2, 2), (16, 16), (16, 21), (17, 19), (100, 100), (256, 300)])
def test_ids_outside_are_skipped(H, k, bad):
    """A vertex with a bad id counts nowhere, and the flag is raised."""
    n = 400
    eptr, pins = nets_of([3] * 200, n, bad)
    part = np.random.default_rng(bad).integers(0, k, n).astype(np.int32)
    part[pins[7]] = bad
    g, _, _ = check(H, eptr, pins, n, k, part)
    with pytest.raises(H.HgError, match="partition id"):
        H.hg_sync_status(g)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 4095, 4096, 4097])
def test_refine_start_with_unaligned_flags(H, n):
    """Eligible flags at an odd address, partitions around the sweep's groups of
    eight: one round of a refinement equals the same from an aligned state."""
    import torch
    eptr, pins = nets_of([min(n, 2)] * 50, n, n)
    k, got = 2, []
    for odd in (0, 1):
        g = H.hg_load_csr(n, eptr, pins, k_max=k)
        sizes = H.state_sizes(n, g.m, k)
        views = {f: torch.empty(c, dtype=t, device="cuda") for f, (t, c) in sizes.items()}
        views["eligible"] = torch.zeros(n + 1, dtype=torch.uint8, device="cuda")[odd:odd + n]
        st = H.State(g, k, np.arange(n, dtype=np.int32) % k, views=views)
        stats = torch.zeros(H.STATS_WORDS, dtype=torch.int64, device="cuda")
        H.hg_refine(g, st, 0.5, 1, stats)
        got.append((st.part.cpu(), st.eligible.cpu(), stats.cpu()))
    assert int(got[0][2][0]) == n                       # every vertex was eligible
    for a, b in zip(*got):
        assert torch.equal(a, b)
