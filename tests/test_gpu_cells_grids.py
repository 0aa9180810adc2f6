"""The one-launch cell list over its grids: keys just below and above 1,024, 2,048, 4,096, 8,192 and
16,384, where the padded scan changes its entries per thread (1 to 16) and where several launches
take over, each with two, four and eight atoms per thread: keys and sorted slots against the host."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

WATER = sy.model_config("water")


# cells per dimension; keys are twice their product
@pytest.mark.parametrize("cells", [(8, 8, 8), (8, 8, 9), (8, 8, 16), (4, 15, 17), (8, 16, 16), (9, 15, 16), (16, 16, 16),
                                   (3, 37, 37), (16, 16, 32), (5, 41, 40)])
@pytest.mark.parametrize("n", [300, 2049, 5001, 8192])
def test_keys_and_slots(cells, n):
    import paper_2604_21441_amd as P
    rng = np.random.default_rng(n)
    box = (np.array(cells) * 5.2 + 0.9).astype(np.float32)
    side = np.maximum(2, np.floor(box / 2.0)).astype(int)
    g = np.stack(np.meshgrid(*[np.arange(k) for k in side], indexing="ij"), -1).reshape(-1, 3)
    pick = rng.permutation(len(g))[:n]
    n = len(pick)
    pos = ((g[pick] + rng.uniform(0.3, 0.7, (n, 3))) * (box / side) + box * rng.integers(-1, 2, (n, 3))).astype(np.float32)
    Z = rng.choice(np.array([1, 8], np.int32), n, p=[0.7, 0.3])
    m = P.NNPModel(WATER, weights=sy.flat_weights(sy.model_weights(WATER, seed=1)))
    m.reserve(int(np.prod(cells)) + n)   # (bins for the whole grid)
    m.compute(torch.from_numpy(pos).cuda(), Z, box)
    torch.cuda.synchronize()
    assert m.status() == 0
    B = P._lib
    key, perm, order, start = (m.read(b) for b in (B.NNP_BUF_KEY, B.NNP_BUF_PERM, B.NNP_BUF_ORDER, B.NNP_BUF_BIN_START))
    assert tuple(m.read(B.NNP_BUF_GRID)[1:]) == cells
    n_bins = int(np.prod(cells))
    ref = orc.cell_list_fp32(pos, orc.species_index(Z, WATER["species"]), 2, box, WATER["rc_rad"])
    assert np.array_equal(key, ref["key"])
    assert np.array_equal(perm, ref["perm"])
    assert np.array_equal(start, ref["bin_start"])
    slot_key = key[perm]
    assert np.array_equal(order, np.lexsort((np.arange(n), slot_key // n_bins, slot_key % n_bins)))
    m.close()
