"""The recount of touched nets at the edges of record and counter widths, queue
lengths and long nets: after every round the state equals a fresh pin count of
the new partition, and the next eligible vertices are the pins of the nets that
a mover touched (whole numbers, exactly)."""
import numpy as np
import pytest

from .test_gpu_counts import H, nets_of  # noqa: F401

pytestmark = pytest.mark.gpu


def _check_round(H, g, before, st, stats, eptr, pins, k, km1_before):
    part = st.part.cpu().numpy()
    fresh = H.State(g, k, part)
    H.hg_compute_pincounts(g, fresh)
    for f in ("phi", "netstate", "block_w", "km1"):
        assert np.array_equal(getattr(st, f).cpu().numpy(), getattr(fresh, f).cpu().numpy()), f
    net = np.repeat(np.arange(eptr.size - 1), np.diff(eptr))
    touched = np.zeros(eptr.size - 1, bool)
    touched[net[(part != before)[pins]]] = True
    eligible = np.zeros(part.size, bool)
    eligible[pins[touched[net]]] = True
    assert np.array_equal(st.eligible.cpu().numpy().astype(bool), eligible)
    (s,) = H.stats_to_dicts(stats)
    assert s["touched_nets"] == touched.sum()
    assert s["touched_pins"] == np.diff(eptr)[touched].sum()
    assert s["km1_delta"] == s["km1_delta_recomputed"] == km1_before - int(st.km1.item())
    return s["approved"]


@pytest.mark.parametrize("how", ["refine", "round", "cached"])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 8, 16, 17, 32, 33, 64, 65, 128, 129, 256])
def test_recount(H, k, how):
    import torch
    n = 3000
    # long nets among short ones, more nets than one block of the sweep holds
    sizes = [1, 2, 255, 256, 257, 63, 64, 65, 1000] + [2 + i % 7 for i in range(1500)]
    eptr, pins = nets_of(sizes, n, k)
    part = np.random.default_rng(k).integers(0, k, n).astype(np.int32)
    w = None if k % 2 else np.random.default_rng(k).integers(1, 5, len(sizes)).astype(np.int32)
    g = H.hg_load_csr(n, eptr, pins, None, w, k_max=k)
    st = H.State(g, k, part)
    stats = torch.zeros(H.STATS_WORDS, dtype=torch.int64, device="cuda")
    H.hg_compute_pincounts(g, st)
    km1 = int(st.km1.item())
    approved = 0
    if how == "refine":
        H.hg_refine(g, st, 0.5, 1, stats)
        approved += _check_round(H, g, part, st, stats, eptr, pins, k, km1)
    else:
        lmax = H.hg_max_block_weight(g, k, 0.5)
        st.eligible.fill_(1)
        if how == "cached":
            cache = H.gain_cache(g, k)
            H.hg_gain_cache_init(g, k, st.part, st.netstate, cache)
        for _ in range(2):
            before, km1 = st.part.cpu().numpy(), int(st.km1.item())
            if how == "cached":
                H.hg_lp_round_cached(g, st, lmax, stats, cache)
                want = H.gain_cache(g, k)
                H.hg_gain_cache_init(g, k, st.part, st.netstate, want)
                for a, b in zip(H.cache_views(g, k, cache), H.cache_views(g, k, want)):
                    assert torch.equal(a, b)
            else:
                H.hg_lp_round(g, st, lmax, stats)
            approved += _check_round(H, g, before, st, stats, eptr, pins, k, km1)
    assert approved > 0


@pytest.mark.parametrize("m", [1, 255, 256, 257, 1023, 1024, 1025, 2049])
@pytest.mark.parametrize("k", [4, 200])
def test_recount_kept_copies(H, m, k):
    """Three rounds in one call (the packed partition follows the moves) equal
    three calls of one round each, at the edges of the sweep's blocks."""
    import torch
    n = 2 * m + 3
    eptr, pins = nets_of([2 + i % 2 for i in range(m)], n, m)
    part = np.random.default_rng(m).integers(0, k, n).astype(np.int32)
    got = []
    for single in (True, False):
        g = H.hg_load_csr(n, eptr, pins, k_max=k)
        st = H.State(g, k, part)
        stats = torch.zeros(3 * H.STATS_WORDS, dtype=torch.int64, device="cuda")
        if single:
            H.hg_compute_pincounts(g, st)
            st.eligible.fill_(1)
            lmax = H.hg_max_block_weight(g, k, 0.5)
            for r in range(3):
                H.hg_lp_round(g, st, lmax, stats[r * H.STATS_WORDS:(r + 1) * H.STATS_WORDS])
        else:
            H.hg_refine(g, st, 0.5, 3, stats)
        got.append([getattr(st, f).cpu() for f in ("part", "phi", "netstate", "block_w",
                                                   "eligible", "km1")] + [stats.cpu()])
    for a, b in zip(*got):
        assert torch.equal(a, b)
