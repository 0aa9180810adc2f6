"""The FP32 network form with the MM potential as an input, which has no bound: atomic energies
and dE/dx against the float64 oracle on the library's own inputs, for potentials from none to far
beyond what the operands' scales provide for, with and without the charge output, in every tiling."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

# As without the MM channel: 22 bits per operand, at most 13 roundings per block of 32 inputs and
# accumulator, six products; an atom beyond the reference potential keeps its bits relative to its
# largest input.
TOL = 1e-5


@pytest.mark.parametrize("kind", ["hcno_mm", "hcno_ee"])
@pytest.mark.parametrize("charge", [0.0, 0.8, 40.0, 1e4, 1e8])
def test_potentials(kind, charge):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    w = sy.model_weights(cfg, seed=2)
    pos, Z = sy.walk_molecule(75, np.random.default_rng(8))
    # one strong charge beside the molecule, so that the potentials of a tile's atoms differ
    mm = np.stack([pos[0], pos.max(0) + 2.0, pos.min(0) - 3.0]).astype(np.float32)
    mm[0] = pos[np.argmax(pos[:, 0])] + np.array([2.0, 0.0, 0.0], np.float32)
    q = np.array([charge, 0.4, -0.4], np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    D = cfg["widths"][0] - 1
    first = None
    for v in (-1, 0, 1, 2, 3, 4, 5, 6, 7):
        m = P.NNPModel(cfg, weights=sy.flat_weights(w))
        m.set_variant("network", v)
        m.compute(t(pos), Z, None, None, t(mm), t(q))
        torch.cuda.synchronize()
        assert m.status() == 0
        whole = m.read(P._lib.NNP_BUF_DEDX)[:, :D]
        first = whole if first is None else first
        assert np.array_equal(whole, first)   # the tilings agree bit for bit
        x = m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :D + 1].astype(np.float64)
        sigma = orc.species_index(Z, cfg["species"])[m.read(P._lib.NNP_BUF_PERM)]
        e, g = orc.mlp_input_grad(x, sigma, w[0], float(cfg["celu_alpha"]))
        if charge >= 1e4:
            assert np.abs(x[:, -1]).max() > 64 * 64
        cols = D + 1 if kind == "hcno_mm" else D   # the charge's own term q joins dE/dphi later
        eg, gg = m.read(P._lib.NNP_BUF_ATOM_ENERGY), m.read(P._lib.NNP_BUF_DEDX)[:, :cols]
        assert np.linalg.norm(eg - e) < TOL * np.linalg.norm(e)
        assert np.linalg.norm(gg - g[:, :cols]) < TOL * np.linalg.norm(g[:, :cols])
        m.close()
