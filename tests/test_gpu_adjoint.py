"""The descriptor adjoint at the edges of its lists: capacities that break the
16-byte alignment of the angular rows, more than 64 radial neighbours, and
lists cut off at their capacity (the call flags NNP_ECAPACITY; the forces are
then those of the cut-off lists, each neighbour receiving the part of a centre
that its own list holds)."""
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


def list_forces(P, m, pos, Z, cfg, box):
    """Forces from the library's own lists and dE/dx, by float64 autograd over the oracle's
    descriptors: a pair whose neighbour's list does not hold the centre acts on the centre only
    (its neighbour is a copy of the atom that no gradient is taken of)."""
    n = len(Z)
    perm = m.read(P._lib.NNP_BUF_PERM)
    cnt = m.read(P._lib.NNP_BUF_NBR_COUNT)
    g = torch.from_numpy(m.read(P._lib.NNP_BUF_DEDX).astype(np.float64))
    sigma = orc.species_index(Z, cfg["species"])[perm]
    x0 = torch.from_numpy(pos[perm].astype(np.float64))
    x = x0.clone().requires_grad_(True)
    both = torch.cat([x, x0])
    rad = m.read(P._lib.NNP_BUF_NBR_RAD)
    held = {(i, j) for i in range(n) for j in rad[i, :cnt[i, 0]]}
    rows = {"rad": rad, "ang": m.read(P._lib.NNP_BUF_NBR_ANG)}
    S = len(cfg["species"])
    total = 0.0
    for kind, col in (("rad", 0), ("ang", 1)):
        I = np.concatenate([np.full(cnt[i, col], i) for i in range(n)]).astype(np.int64)
        J = np.concatenate([rows[kind][i, :cnt[i, col]] for i in range(n)]).astype(np.int64)
        J = np.array([j if (j, i) in held else n + j for i, j in zip(I, J)], dtype=np.int64)
        d = orc.descriptors(both, np.concatenate([sigma, sigma]), cfg, box=box, centres=np.arange(n), pairs_rad=(I, J))
        part = slice(0, 16 * S) if kind == "rad" else slice(16 * S, d.shape[1])
        total = total + (d[:, part] * g[:, :d.shape[1]][:, part]).sum()
    grad, = torch.autograd.grad(total, x)
    F = np.empty((n, 3))
    F[perm] = -grad.numpy()
    return F


def run(m, pos, Z, box):
    E, F, _ = m.compute(torch.from_numpy(pos).cuda(), Z, box)
    torch.cuda.synchronize()
    return F.cpu().numpy()


# FP32 terms of about 60 pairs and 130 triplets per atom summed in FP64: the
# error stays within the FP32 form's 1e-5, as for the forces as a whole
TOL = 1e-5


@pytest.mark.parametrize("max_rad,max_ang", [(128, 64), (128, 63), (127, 62), (1024, 256), (72, 28)])
def test_capacities(P, max_rad, max_ang):
    """Row pitches with and without 16-byte alignment, up to the largest capacities."""
    pos, Z, box = sy.water_box(216, 18.63, seed=3)
    m = P.NNPModel(WATER, weights=sy.flat_weights(sy.model_weights(WATER, seed=1)))
    m.reserve(len(Z), max_rad_nbr=max_rad, max_ang_nbr=max_ang)
    F = run(m, pos, Z, box)
    assert m.status() == 0
    ref = list_forces(P, m, pos, Z, WATER, box)
    assert np.linalg.norm(F - ref) < TOL * np.linalg.norm(ref)
    m.close()


@pytest.mark.parametrize("spacing", [1.0, 1.25])
def test_dense_molecule(P, spacing):
    """A jittered lattice cut to a ball: up to 128 < nr radial neighbours (two geometry passes and
    more), about 100 angular ones, four elements."""
    rng = np.random.default_rng(5)
    g = np.stack(np.meshgrid(*[np.arange(-6, 7)] * 3, indexing="ij"), -1).reshape(-1, 3) * spacing
    pos = g[np.linalg.norm(g, axis=1) < 5.0]
    pos = (pos + rng.uniform(-0.05, 0.05, pos.shape)).astype(np.float32)
    Z = rng.choice(np.array([1, 6, 7, 8], np.int32), len(pos))
    m = P.NNPModel(HCNO, weights=sy.flat_weights(sy.model_weights(HCNO, seed=1)))
    m.reserve(len(Z), max_rad_nbr=640, max_ang_nbr=256)
    F = run(m, pos, Z, None)
    assert m.status() == 0
    assert m.read(P._lib.NNP_BUF_NBR_COUNT)[:, 0].max() > 128
    ref = list_forces(P, m, pos, Z, HCNO, None)
    assert np.linalg.norm(F - ref) < TOL * np.linalg.norm(ref)
    m.close()


@pytest.mark.parametrize("max_rad,max_ang", [(40, 64), (128, 11), (33, 9)])
def test_cut_off_lists(P, max_rad, max_ang):
    """Overflowing lists set the status and give the forces of the cut-off lists; after the status
    is read, a call with room again gives the ordinary ones."""
    pos, Z, box = sy.water_box(125, 15.52, seed=4)
    m = P.NNPModel(WATER, weights=sy.flat_weights(sy.model_weights(WATER, seed=1)))
    m.reserve(len(Z), max_rad_nbr=max_rad, max_ang_nbr=max_ang)
    F = run(m, pos, Z, box)
    F2 = run(m, pos, Z, box)
    ref = list_forces(P, m, pos, Z, WATER, box)
    assert m.status() == P._lib.NNP_ECAPACITY
    assert np.linalg.norm(F - ref) < TOL * np.linalg.norm(ref)
    assert np.allclose(F, F2, rtol=0, atol=1e-6 * np.abs(F).max())
    m.reserve(len(Z), max_rad_nbr=128, max_ang_nbr=64)
    F = run(m, pos, Z, box)
    assert m.status() == 0
    ref = list_forces(P, m, pos, Z, WATER, box)
    assert np.linalg.norm(F - ref) < TOL * np.linalg.norm(ref)
    m.close()
