"""Rounds without threshold and tile-scan launches (one small graph) against the
batched rounds, which have them: the same state and records, bit for bit, at the
edges of tiles, of the rule's sizes and block counts, with budgets that cut most
blocks, weighted vertices among them."""
import numpy as np
import pytest

import synth

from .test_gpu_batch import H, _members, _snapshot  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(1, 2), (2, 2), (511, 3), (512, 16), (513, 17), (2047, 2),
                                 (2049, 16), (60000, 5), (131072, 16), (131073, 16),
                                 (131071, 2)])
@pytest.mark.parametrize("unit", [True, False])
@pytest.mark.parametrize("eps", [0.002, 0.5])
def test_brief_rounds_equal_batched_rounds(H, n, k, unit, eps):
    import torch
    inst = synth.random_power_law(7 * n + k, n, max(n - 3, 1), k, hi=min(n, 12), lo=min(n, 2),
                                  unit=unit, eps=eps, rounds=4)
    got = []
    for batched in (False, True):
        (mb,) = _members(H, [inst], 4)
        if batched:
            b = H.hg_batch_create([mb])
            H.hg_batch_refine(b, 4)
            torch.cuda.synchronize()
            b.free()
        else:
            H.hg_refine(mb.g, mb.st, inst.eps, 4, mb.stats)
        got.append(_snapshot(mb))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [98304, 98305])
@pytest.mark.parametrize("k", [2, 16])
def test_largest_brief_rounds_equal_batched_rounds(H, n, k):
    test_brief_rounds_equal_batched_rounds(H, n, k, False, 0.01)


@pytest.mark.parametrize("n", [131072, 131073])
@pytest.mark.parametrize("k", [8, 9])
def test_edge_of_block_counts_equals_batched_rounds(H, n, k):
    test_brief_rounds_equal_batched_rounds(H, n, k, True, 0.01)
