"""Members shared over grid rows in the networks with the MM potential (416 inputs), whose operands'
scales depend on the atom's potential, and in the BF16 form of every width."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# As for one network (six products of 22-bit operands), the average adding FP32 roundings
@pytest.mark.parametrize("members", [2, 3, 8])
@pytest.mark.parametrize("charge", [0.0, 0.8, 1e4])
def test_potential(members, charge):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("hcno_mm")
    w = sy.model_weights(cfg, seed=2, n_members=members)
    pos, Z = sy.walk_molecule(75, np.random.default_rng(8))
    mm = np.stack([pos[np.argmax(pos[:, 0])] + np.float32([2.0, 0.0, 0.0]), pos.max(0) + 2.0,
                   pos.min(0) - 3.0]).astype(np.float32)
    q = np.array([charge, 0.4, -0.4], np.float32)
    m = P.NNPModel(cfg, weights=sy.flat_weights(w), n_members=members)
    for _ in range(2):
        E, F, _ = m.compute(t(pos), Z, None, None, t(mm), t(q))
    torch.cuda.synchronize()
    assert m.status() == 0 and m.variants()["network"] == 5
    D = cfg["widths"][0]
    x = m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :D].astype(np.float64)
    sigma = orc.species_index(Z, cfg["species"])[m.read(P._lib.NNP_BUF_PERM)]
    each = [orc.mlp_input_grad(x, sigma, one, float(cfg["celu_alpha"])) for one in w]
    e, g = (sum(part) / members for part in zip(*each))
    eg, gg = m.read(P._lib.NNP_BUF_ATOM_ENERGY), m.read(P._lib.NNP_BUF_DEDX)[:, :D]
    assert np.linalg.norm(eg - e) < 1e-5 * np.linalg.norm(e)
    assert np.linalg.norm(gg - g) < 1e-5 * np.linalg.norm(g)
    assert abs(E.item() - eg.astype(np.float64).sum()) < 1e-9 * np.abs(eg).sum()
    m.close()


# The same BF16 products with the average taken in another order (FP32 roundings of 2^-24 each)
@pytest.mark.parametrize("kind,members", [("water", 2), ("water", 5), ("hcno", 3), ("hcno_mm", 4)])
def test_bf16(kind, members):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    w = sy.flat_weights(sy.model_weights(cfg, seed=2, n_members=members))
    extra = {}
    box = None
    if kind == "water":
        pos, Z, box = sy.water_box(90, 13.9, seed=6)
    else:
        pos, Z = sy.walk_molecule(75, np.random.default_rng(8))
    if kind == "hcno_mm":
        extra = {"mm_pos": t(pos + np.float32([0.0, 0.0, 9.0])), "mm_q": t(np.linspace(-0.6, 0.6, len(Z)).astype(np.float32))}
    m = P.NNPModel(cfg, weights=w, precision="bf16", n_members=members)
    got = []
    for pin in (-1, 1):   # shared over rows, and one workgroup walking all members
        m.set_variant("network", pin)
        E, F, _ = m.compute(t(pos), Z, box, **extra)
        torch.cuda.synchronize()
        assert m.status() == 0
        got.append([m.read(P._lib.NNP_BUF_ATOM_ENERGY).astype(np.float64), m.read(P._lib.NNP_BUF_DEDX).astype(np.float64),
                    E.cpu().numpy(), F.cpu().numpy()])
    for a, b, tol in zip(*got, (1e-6, 1e-6, 1e-6, 1e-5)):
        assert np.linalg.norm(a - b) < tol * np.linalg.norm(b), np.linalg.norm(a - b) / np.linalg.norm(b)
    m.close()
