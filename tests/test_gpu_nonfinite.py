"""Inputs and weights that make a descriptor, an MM potential or an activation NaN: the energy is
NaN and the status NNP_ENONFINITE, in every network tiling and in both forms, and other systems of
a batch keep their results."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu

VARIANTS = (-1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9)


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def flagged(P, m, E, *forces):
    torch.cuda.synchronize()
    assert m.status() == P._lib.NNP_ENONFINITE
    assert np.isnan(E.cpu().numpy()).any()
    assert all(not np.isfinite(f.cpu().numpy()).all() for f in forces)
    assert m.status() == 0   # (reading clears it)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("members", [1, 4])
def test_coincident_atoms(prec, members):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("water")
    pos, Z, box = sy.water_box(64, 12.42, seed=0)
    bad = pos.copy()
    bad[7] = bad[3]
    w = sy.flat_weights(sy.model_weights(cfg, seed=1, n_members=members))
    m = P.NNPModel(cfg, weights=w, precision=prec, n_members=members)
    for v in VARIANTS:
        m.set_variant("network", v)
        E, F, _ = m.compute(t(bad), Z, box)
        flagged(P, m, E, F)
        E, F, _ = m.compute(t(pos), Z, box)
        torch.cuda.synchronize()
        assert m.status() == 0 and torch.isfinite(E).all() and torch.isfinite(F).all()
    m.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_one_system_of_a_batch(prec):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("hcno")
    pos, Z, off = sy.walk_batch(6, seed=5)
    bad = pos.copy()
    bad[off[2] + 1] = bad[off[2]]
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=1)), precision=prec)
    for v in VARIANTS[:8]:
        m.set_variant("network", v)
        E0, F0 = m.compute_batch(t(pos), Z, off)
        assert m.status() == 0
        E, F = m.compute_batch(t(bad), Z, off)
        flagged(P, m, E[2:3], F[off[2]:off[3]])
        for s in (0, 1, 3, 4, 5):
            assert E[s].item() == E0[s].item()
            assert torch.allclose(F[off[s]:off[s + 1]], F0[off[s]:off[s + 1]], rtol=1e-12, atol=1e-12)
    m.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("kind", ["hcno_mm", "hcno_ee"])
@pytest.mark.parametrize("fault", ["charge on an atom", "NaN charge", "infinite charge"])
def test_mm_potential(prec, kind, fault):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    pos, Z = sy.walk_molecule(30, np.random.default_rng(4))
    mm = (pos + np.float32([0.0, 0.0, 8.0])).astype(np.float32)
    q = np.linspace(-0.5, 0.5, len(Z)).astype(np.float32)
    if fault == "charge on an atom":
        mm[5] = pos[3]
    else:
        q[5] = np.nan if fault == "NaN charge" else np.inf
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=2)), precision=prec)
    for v in VARIANTS[:9]:
        m.set_variant("network", v)
        E, F, Fmm = m.compute(t(pos), Z, None, None, t(mm), t(q))
        flagged(P, m, E, F)
    m.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("layer,what", [(0, "bias"), (1, "bias"), (2, "bias"), (3, "bias"), (0, "weight"),
                                        (1, "weight"), (2, "weight"), (3, "weight")])
def test_nan_parameter(prec, layer, what):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("water")
    pos, Z, box = sy.water_box(64, 12.42, seed=0)
    w = sy.model_weights(cfg, seed=1)
    W, b = (a.copy() for a in w[0][1][layer])
    # (the all-ones payload is the one that rounding to BF16 could carry over)
    nan = np.array([0x7FFFFFFF], np.uint32).view(np.float32)[0]
    if what == "bias":
        b[-1] = nan
    else:
        W[-1, -1] = nan
    w[0][1][layer] = (W, b)
    m = P.NNPModel(cfg, weights=sy.flat_weights(w), precision=prec)
    for v in VARIANTS:
        m.set_variant("network", v)
        E, F, _ = m.compute(t(pos), Z, box)
        flagged(P, m, E, *([F] if (layer, what) != (3, "bias") else []))
    m.close()
