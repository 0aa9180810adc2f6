"""The sum of the atomic energies: an FP32 network's weights are constants, so
an error of theirs does not average out over atoms as the accumulators'
roundings do.  The mean signed error of the atomic energies against the
float64 oracle on the library's own descriptors."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    import paper_2604_21441_amd as P
    return P


# FP32 products of unrounded FP32 weights leave 1e-9 to 5e-9 (water) on these
# systems, from the FP32 activations; twice the largest.  Independent roundings
# of 1e-7 an atom add 3e-9 over 1,500 atoms.
BOUND = 1e-8


@pytest.mark.parametrize("kind,seed", [("water", 1), ("water", 2), ("water", 5), ("hcno", 2)])
def test_mean_error(P, kind, seed):
    cfg = sy.model_config(kind)
    if kind == "water":
        pos, Z, box = sy.water_box(500, 12.42 * (500 / 64) ** (1 / 3), seed=seed)
    else:
        (pos, Z), box = sy.walk_molecule(1500, np.random.default_rng(8 + seed)), None
    w = sy.model_weights(cfg, seed=seed)
    for v in (-1, 0, 2, 5, 7):
        m = P.NNPModel(cfg, weights=sy.flat_weights(w))
        m.set_variant("network", v)
        m.compute(torch.from_numpy(pos).cuda(), Z, box)
        assert m.status() == 0
        x = m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, : cfg["widths"][0]].astype(np.float64)
        sigma = orc.species_index(Z, cfg["species"])[m.read(P._lib.NNP_BUF_PERM)]
        e, _ = orc.mlp_input_grad(x, sigma, w[0], float(cfg["celu_alpha"]))
        d = m.read(P._lib.NNP_BUF_ATOM_ENERGY).astype(np.float64) - e
        m.close()
        assert abs(d.mean()) < BOUND, (v, d.mean())
