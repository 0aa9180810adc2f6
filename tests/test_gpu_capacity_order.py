"""Reserved capacities with fewer radial than angular neighbours, and lists that fit: the force
contributions have a row of max_ang entries per atom whichever capacity is the larger, so the last
atoms' rows must not reach the arrays behind them (totals, energy partials, descriptors)."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


# FP32 pair and triplet terms summed in FP64: the FP32 form's 1e-5 of the forces, 1e-6 per atom
@pytest.mark.parametrize("kind,max_rad,max_ang", [("hcno", 32, 64), ("hcno", 32, 0), ("hcno", 32, 255),
                                                  ("water", 40, 256), ("pairs", 32, 64), ("batch", 80, 160)])
def test_forces(kind, max_rad, max_ang):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("water" if kind == "water" else "hcno")
    off = None
    if kind == "water":       # a drop, open boundaries
        pos, Z, _ = sy.water_box(8, 8.0, seed=3)
    elif kind == "batch":
        pos, Z, off = sy.walk_batch(6, seed=5)
    else:
        pos, Z = sy.walk_molecule(30, np.random.default_rng(12))
    off = np.array([0, len(Z)]) if off is None else off
    w = sy.model_weights(cfg, seed=1)
    m = P.NNPModel(cfg, weights=sy.flat_weights(w))
    m.reserve(len(Z), max_systems=len(off) - 1, max_rad_nbr=max_rad, max_ang_nbr=max_ang)
    d = torch.from_numpy(pos).cuda()
    for _ in range(2):
        if kind == "batch":
            E, F = m.compute_batch(d, Z, off)
        elif kind == "pairs":
            I, J = orc.neighbour_pairs(pos, 5.6, None)
            pairs = np.stack([I[I < J], J[I < J]], 1).astype(np.int32)
            E, F, _ = m.compute_pairs(d, torch.from_numpy(pairs).cuda(), Z)
        else:
            E, F, _ = m.compute(d, Z)
    torch.cuda.synchronize()
    assert m.status() == 0   # (both lists fit)
    for s, (a, b) in enumerate(zip(off[:-1], off[1:])):
        ref = orc.evaluate(pos[a:b], Z[a:b], cfg, w)
        assert abs(E[s].item() - ref["E"]) < 1e-6 * (b - a)
        assert np.linalg.norm(F[a:b].cpu().numpy() - ref["F"]) < 1e-5 * np.linalg.norm(ref["F"])
    m.close()
