"""The one-launch cell list at its sizes' edges (one to eight atoms per thread, one to eight
workgroups) and on both sides of the size where three launches take over: keys equal to those of
the whole system, slots a stable sort by key, the visiting order bin by bin."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu

WATER = sy.model_config("water")
SIZES = [1, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193]


@pytest.fixture(scope="module")
def system():
    import paper_2604_21441_amd as P
    pos, Z, box = sy.water_box(3000, 12.42 * (3000 / 64) ** (1 / 3), seed=9)
    m = P.NNPModel(WATER, weights=sy.flat_weights(sy.model_weights(WATER, seed=1)))
    m.compute(torch.from_numpy(pos).cuda(), Z, box)
    assert m.status() == 0
    return P, pos, Z, box, m, m.read(P._lib.NNP_BUF_KEY).copy()


@pytest.mark.parametrize("n", SIZES)
def test_sorted_slots(system, n):
    P, pos, Z, box, m, keys = system
    idx = np.random.default_rng(n).permutation(len(Z))[:n].astype(np.int32)
    m.compute(torch.from_numpy(pos).cuda(), Z, box, idx)
    assert m.status() == 0
    B = P._lib
    key, perm, order, start = (m.read(b) for b in (B.NNP_BUF_KEY, B.NNP_BUF_PERM, B.NNP_BUF_ORDER, B.NNP_BUF_BIN_START))
    assert np.array_equal(key, keys[idx])
    assert np.array_equal(perm, np.argsort(key, kind="stable"))
    n_bins = (len(start) - 1) // 2
    assert np.array_equal(start, np.searchsorted(key[perm], np.arange(2 * n_bins + 1)))
    slot_key = key[perm]
    assert np.array_equal(order, np.lexsort((np.arange(n), slot_key // n_bins, slot_key % n_bins)))
