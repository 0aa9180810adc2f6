"""The FP32 network form on FP16 operand pairs: atomic energies and dE/dx
against the float64 oracle on the library's own descriptors, over weights of
very different magnitudes (the power-of-two scales of the operands follow from
them), the largest list capacities (the loosest bounds on the activations),
every tiling and ensembles."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

WATER = sy.model_config("water")
HCNO = sy.model_config("hcno")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    import paper_2604_21441_amd as P
    return P


def scaled(cfg, factors, members=1):
    """Weights with layer l's matrix and bias multiplied by factors[l]."""
    w = sy.model_weights(cfg, seed=2, n_members=members)
    return [[[((W * f).astype(np.float32), (b * f).astype(np.float32)) for (W, b), f in zip(layers, factors)]
             for layers in species] for species in w]


# Each operand carries 22 bits and an accumulator takes at most 13 FP32
# roundings per K block of 32: relative to the sum of magnitudes of a row
# (about sqrt(K) times the result) an error near 2^-22, through six products.
# The FP32 form's stated 1e-5 leaves a factor of a few for cancellation.
TOL = 1e-5


def check(P, m, Z, cfg, w):
    perm = m.read(P._lib.NNP_BUF_PERM)
    D = cfg["widths"][0]
    x = m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :D].astype(np.float64)
    sigma = orc.species_index(Z, cfg["species"])[perm]
    alpha = float(cfg["celu_alpha"])
    each = [orc.mlp_input_grad(x, sigma, member, alpha) for member in w]
    e, g = (sum(part) / len(w) for part in zip(*each))
    eg = m.read(P._lib.NNP_BUF_ATOM_ENERGY)
    gg = m.read(P._lib.NNP_BUF_DEDX)[:, :D]
    assert np.linalg.norm(eg - e) < TOL * np.linalg.norm(e), np.linalg.norm(eg - e) / np.linalg.norm(e)
    assert np.linalg.norm(gg - g) < TOL * np.linalg.norm(g), np.linalg.norm(gg - g) / np.linalg.norm(g)


FACTORS = [(1, 1, 1, 1), (1e3, 1e-3, 1, 1), (1e-4, 1, 1e4, 1e-6), (1, 1e5, 1e-5, 1e3), (1e-3, 1e-3, 1e-3, 1e-3)]


@pytest.mark.parametrize("factors", FACTORS)
@pytest.mark.parametrize("caps", [(0, 0), (1024, 256)])
def test_weight_magnitudes(P, factors, caps):
    pos, Z, box = sy.water_box(70, 12.8, seed=6)   # 70 O and 140 H: ragged tiles
    w = scaled(WATER, factors)
    m = P.NNPModel(WATER, weights=sy.flat_weights(w))
    m.reserve(len(Z), max_rad_nbr=caps[0], max_ang_nbr=caps[1])
    m.compute(torch.from_numpy(pos).cuda(), Z, box)
    assert m.status() == 0
    check(P, m, Z, WATER, w)
    m.close()


@pytest.mark.parametrize("kind,members", [("water", 1), ("water", 3), ("hcno", 1)])
def test_tilings(P, kind, members):
    cfg = WATER if kind == "water" else HCNO
    w = scaled(cfg, (1, 1, 1, 1), members)
    if kind == "water":
        pos, Z, box = sy.water_box(70, 12.8, seed=6)
    else:
        pos, Z = sy.walk_molecule(75, np.random.default_rng(8))
        box = None
    for v in (-1, 0, 1, 2, 3, 4, 5, 6, 7):
        m = P.NNPModel(cfg, weights=sy.flat_weights(w), n_members=members)
        m.set_variant("network", v)
        m.compute(torch.from_numpy(pos).cuda(), Z, box)
        assert m.status() == 0
        check(P, m, Z, cfg, w)
        m.close()
