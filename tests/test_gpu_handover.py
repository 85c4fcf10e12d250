"""What one call leaves in a handle's workspace for the next: calls of every kind in
turn on one handle against each on a fresh one, refinement with its phases timed
against untimed, and rounds of one refinement that hand over more than a plain round
does (a budget that ends inside the highest gain bucket, an id out of range)."""
import numpy as np
import pytest

from oracle import oracle as O
import synth

from .test_gpu_batch import H, _hub_instance, _snapshot  # noqa: F401
from .test_gpu_fullsize import _overflow_instance
from .test_gpu_parity import _check_state, _oracle_hg

pytestmark = pytest.mark.gpu

K_MAX = 64


def _load(H, inst):
    return H.hg_load_csr(inst.n, inst.eptr, inst.pins, inst.c, inst.w, k_max=K_MAX)


def _call(H, g, inst, how, k, rounds=3):
    """One call from a start of its own; all it writes."""
    import torch
    st = H.State(g, k, np.random.default_rng(k).integers(0, k, inst.n).astype(np.int32))
    st.eligible.fill_(1)
    stats = torch.zeros(rounds * H.STATS_WORDS, dtype=torch.int64, device="cuda")
    lmax = H.hg_max_block_weight(g, k, inst.eps)
    mb = H.Member(g, st, inst.eps, stats)
    extra = []
    if how in ("refine", "graph", "timed"):
        H.hg_timing_enable(g, how == "timed")
        H.hg_refine(g, st, inst.eps, rounds, stats, use_graph=how == "graph")
        if how == "timed":
            assert H.hg_timing_collect(g)[1] == rounds
            H.hg_timing_enable(g, False)
    elif how in ("round", "noalloc"):
        H.hg_compute_pincounts(g, st)
        (H.hg_lp_round if how == "round" else H.hg_lp_round_noalloc)(g, st, lmax, stats)
    elif how == "cached":
        cache = H.gain_cache(g, k)
        H.hg_refine_cached(g, st, inst.eps, rounds, stats, cache)
        extra = list(H.cache_views(g, k, cache))
    elif how == "exact":
        H.hg_refine_exact(g, st, inst.eps, rounds, stats, H.moves_workspace(g, k))
    elif how == "rebalance":
        H.hg_compute_pincounts(g, st)
        H.hg_rebalance(g, st, lmax, 2, stats, H.rebalance_workspace(g, k))
    else:
        b = H.hg_batch_create([mb])
        H.hg_batch_refine(b, rounds)
        torch.cuda.synchronize()
        b.free()
    torch.cuda.synchronize()
    H.hg_sync_status(g)
    return _snapshot(mb) + [x.cpu().numpy() for x in extra]


# Block counts on both sides of the brief rounds' limit, of the packed partition's and
# of the views', each kind after each other at least once.
TURNS = [("refine", 16), ("round", 17), ("refine", 2), ("cached", 64), ("graph", 16),
         ("refine", 64), ("noalloc", 3), ("refine", 33), ("timed", 16), ("round", 2),
         ("batch", 8), ("refine", 17), ("exact", 5), ("refine", 8), ("rebalance", 4),
         ("timed", 64), ("refine", 16), ("batch", 64), ("graph", 2), ("cached", 16),
         ("round", 16), ("refine", 16)]


@pytest.mark.parametrize("kind", ["light", "heavy"])
def test_calls_in_turn_on_one_handle(H, kind):
    if kind == "light":
        inst = synth.random_power_law(41, 9000, 8500, K_MAX, hi=14, unit=False, eps=0.02)
    else:
        inst = _hub_instance(8, 6000, 5000, K_MAX, 400, True)
    fresh = {}
    g = _load(H, inst)
    for turn, (how, k) in enumerate(TURNS):
        if (how, k) not in fresh:
            other = _load(H, inst)
            fresh[how, k] = _call(H, other, inst, how, k)
            other.free()
        got = _call(H, g, inst, how, k)
        assert len(got) == len(fresh[how, k])
        for a, b in zip(got, fresh[how, k]):
            assert np.array_equal(a, b), (turn, how, k)
    for k in (2, 16, 64):
        want = fresh["refine", k]
        for how in ("timed", "graph", "batch"):
            if (how, k) in fresh:
                for a, b in zip(fresh[how, k], want):
                    assert np.array_equal(a, b), (how, k)


@pytest.mark.parametrize("use_graph", [False, True])
def test_rounds_of_overflowing_budgets(H, use_graph):
    import torch
    R = 4
    inst = _overflow_instance()
    h = _oracle_hg(inst)
    lmax = O.lmax(O.total_vertex_weight(h), 2, inst.eps)
    g = H.hg_load_csr(inst.n, inst.eptr, inst.pins, inst.c, inst.w, k_max=2)
    assert H.hg_get_info(g)["heavy_vertices"] == 7
    part_o, stats_o, km1_o = O.refine(h, 2, lmax, R, inst.part)
    for _ in range(2):
        st = H.State(g, 2, inst.part)
        stats = torch.zeros(R * H.STATS_WORDS, dtype=torch.int64, device="cuda")
        H.hg_refine(g, st, inst.eps, R, stats, use_graph=use_graph)
        torch.cuda.synchronize()
        got = H.stats_to_dicts(stats)
        for r in range(R):
            assert got[r].pop("km1_delta_recomputed") == got[r]["km1_delta"]
            assert got[r] == stats_o[r], r
        assert np.array_equal(st.part.cpu().numpy(), part_o)
        assert int(st.km1.item()) == km1_o
        _check_state(H, g, st, h, 2, part_o)
    H.hg_sync_status(g)


@pytest.mark.parametrize("k", [2, 8, 16, 17, 64])
def test_refine_with_an_id_out_of_range_equals_rounds(H, k):
    import torch
    R = 3
    inst = synth.random_power_law(50 + k, 5000, 4800, k, hi=12, unit=False, eps=0.05)
    part = inst.part.copy()
    part[1234] = k
    got = []
    for refine in (True, False):
        g = H.hg_load_csr(inst.n, inst.eptr, inst.pins, inst.c, inst.w, k_max=k)
        st = H.State(g, k, part)
        stats = torch.zeros(R * H.STATS_WORDS, dtype=torch.int64, device="cuda")
        if refine:
            H.hg_refine(g, st, inst.eps, R, stats, use_graph=False)
        else:
            H.hg_compute_pincounts(g, st)
            st.eligible.fill_(1)
            lmax = H.hg_max_block_weight(g, k, inst.eps)
            for r in range(R):
                H.hg_lp_round(g, st, lmax, stats[r * H.STATS_WORDS:(r + 1) * H.STATS_WORDS])
        torch.cuda.synchronize()
        with pytest.raises(H.HgError, match="partition id"):
            H.hg_sync_status(g)
        got.append(_snapshot(H.Member(g, st, inst.eps, stats)))
    assert H.stats_to_dicts(torch.as_tensor(got[0][-1]))[0]["approved"] > 0
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert got[0][0][1234] == k
