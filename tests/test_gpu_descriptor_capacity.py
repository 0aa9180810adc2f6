"""The default descriptor kernel of large two-element systems by the angular capacity, which sizes
its LDS: four pooled atoms per wavefront up to 96 entries, rows of lanes beyond, up to the largest
capacity, with the same descriptors as one wavefront per atom."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu


# FP32 sums of some hundred terms of one sign in another order: 5e-6 of a row's norm
@pytest.mark.parametrize("max_ang,variant", [(64, 4), (96, 4), (97, 1), (256, 1)])
def test_choice(max_ang, variant):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("water")
    n_mol = 24 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    pos, Z, box = sy.water_box(n_mol, 12.42 * (n_mol / 64) ** (1 / 3), seed=3)
    d = torch.from_numpy(pos).cuda()
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=1)))
    m.reserve(len(Z), max_ang_nbr=max_ang)
    rows = []
    for pin in (-1, 4, 0):
        m.set_variant("descriptor", pin)
        m.compute(d, Z, box)
        torch.cuda.synchronize()
        assert m.status() == 0
        if pin < 0:
            assert m.variants()["descriptor"] == variant
        rows.append(m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :128].copy())
    for r in rows[:2]:
        err = np.linalg.norm(r - rows[2], axis=1)
        assert np.all(err <= 5e-6 * np.linalg.norm(rows[2], axis=1)), err.max()
    m.close()
