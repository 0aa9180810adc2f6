"""Ensembles whose members are shared over grid rows (few tiles): members that do not divide
evenly, two and four rows, both tile sizes, batches, and a workspace too small for the rows'
sums -- atomic energies, total energy and dE/dx against the float64 oracle on the library's own
descriptors."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

# As for one network (six products of 22-bit operands), the average over members adding FP32
# roundings of 2^-24
TOL = 1e-5


@pytest.mark.parametrize("kind,n_mol,members,max_rad", [("water", 64, 2, 0), ("water", 64, 3, 0), ("water", 90, 5, 0),
                                                        ("water", 90, 8, 0), ("water", 90, 8, 42),
                                                        ("water", 1500, 5, 0), ("hcno", 0, 3, 0),
                                                        ("hcno", 40, 5, 0)])
def test_average(kind, n_mol, members, max_rad):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    w = sy.model_weights(cfg, seed=2, n_members=members)
    box = off = None
    if kind == "water":
        pos, Z, box = sy.water_box(n_mol, 12.6 * (n_mol / 64) ** (1 / 3), seed=6)
    elif n_mol:
        pos, Z, off = sy.walk_batch(n_mol, seed=7)
    else:
        pos, Z = sy.walk_molecule(75, np.random.default_rng(8))
    m = P.NNPModel(cfg, weights=sy.flat_weights(w), n_members=members)
    if max_rad:
        m.reserve(len(Z), max_rad_nbr=max_rad)
    d = torch.from_numpy(pos).cuda()
    for _ in range(2):
        E = (m.compute_batch(d, Z, off) if off is not None else m.compute(d, Z, box))[0]
    torch.cuda.synchronize()
    assert m.status() == (P._lib.NNP_ECAPACITY if max_rad else 0)   # (cut-off lists are lists all the same)
    D = cfg["widths"][0]
    perm = m.read(P._lib.NNP_BUF_PERM)
    x = m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :D].astype(np.float64)
    sigma = orc.species_index(Z, cfg["species"])[perm]
    each = [orc.mlp_input_grad(x, sigma, one, float(cfg["celu_alpha"])) for one in w]
    e, g = (sum(part) / members for part in zip(*each))
    eg, gg = m.read(P._lib.NNP_BUF_ATOM_ENERGY), m.read(P._lib.NNP_BUF_DEDX)[:, :D]
    assert np.linalg.norm(eg - e) < TOL * np.linalg.norm(e)
    assert np.linalg.norm(gg - g) < TOL * np.linalg.norm(g)
    if off is None:
        assert abs(E.sum().item() - eg.astype(np.float64).sum()) < 1e-9 * np.abs(eg).sum()
    else:
        slot = np.empty(len(Z))
        slot[perm] = eg
        assert np.allclose(E.cpu().numpy(), np.add.reduceat(slot, off[:-1]), rtol=0, atol=1e-9 * np.abs(eg).sum())
    m.close()
