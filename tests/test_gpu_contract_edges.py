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
