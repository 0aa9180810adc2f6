"""The cell neighbour kernel (variants 1 to 3) against the one-wavefront-per-atom
kernel, bit for bit: lists, species segments (through the descriptors, which sum
each segment in list order) and the overflow status, where its shortcut could go
wrong: three and four cells per dimension, flat boxes, atoms moved by many box
lengths, atoms exactly on a cutoff, cells with more candidates than the kernel's
registers hold, and lists at their capacity."""
import numpy as np
import pytest
import torch

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


def gas(rng, box, density, species, dmin=0.8):
    """Uniformly random atoms, jittered off a lattice of spacing dmin or more."""
    n = np.maximum(1, np.floor(np.asarray(box) / max(dmin, density ** (-1 / 3)))).astype(int)
    g = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 3)
    pos = (g + rng.uniform(0.25, 0.75, g.shape)) * (np.asarray(box) / n)
    return pos.astype(np.float32), rng.choice(np.array(species, np.int32), len(pos))


def inputs(name):
    rng = np.random.default_rng(11)
    if name == "three_cells":
        return (*gas(rng, [16.5] * 3, 0.1, (1, 8)), np.full(3, 16.5, np.float32), WATER)
    if name == "three_cells_tight":      # cells no longer than the cutoff: the atom kernel runs
        return (*gas(rng, [15.602] * 3, 0.1, (1, 8)), np.full(3, 15.602, np.float32), WATER)
    if name == "flat":
        box = [16.1, 21.3, 47.9]
        return (*gas(rng, box, 0.1, (1, 8)), np.array(box, np.float32), WATER)
    if name in ("moved", "far"):         # whole box lengths, to 10^2 and 10^5 A
        pos, Z, box = sy.water_box(216, 21.5, seed=2)
        k = rng.integers(-5, 6, pos.shape) * (1 if name == "moved" else 1000)
        return (pos + k * box).astype(np.float32), Z, box, WATER
    if name == "on_cutoff":              # lattice spacings that put many pairs on a cutoff
        g = np.stack(np.meshgrid(*[np.arange(12)] * 3, indexing="ij"), -1).reshape(-1, 3)
        pos = (g * np.float32(5.2 / 3)).astype(np.float32)
        return pos, rng.choice(np.array([1, 8], np.int32), len(pos)), np.full(3, 20.8, np.float32), WATER
    if name == "four_elements":
        return (*gas(rng, [22.0, 27.0, 31.0], 0.1, (1, 6, 7, 8)), np.array([22.0, 27.0, 31.0], np.float32), HCNO)
    if name == "missing_species":        # no atom of the first and the third species
        return (*gas(rng, [22.0] * 3, 0.1, (6, 8)), np.full(3, 22.0, np.float32), HCNO)
    if name == "dense":                  # about 1,000 candidates per cell, beyond the registers
        return (*gas(rng, [21.0] * 3, 0.3, (1, 6, 7, 8)), np.full(3, 21.0, np.float32), HCNO)
    raise KeyError(name)


def lists(P, cfg, pos, Z, box, variant, caps):
    m = P.NNPModel(cfg, seed=1)
    m.reserve(len(Z), max_rad_nbr=caps[0], max_ang_nbr=caps[1])
    m.set_variant("neighbours", variant)
    m.compute(torch.from_numpy(pos).cuda(), Z, box)
    torch.cuda.synchronize()
    ran = m.variants()["neighbours"]
    out = [m.status(), m.read(P._lib.NNP_BUF_NBR_COUNT)]
    for which, col in ((P._lib.NNP_BUF_NBR_RAD, 0), (P._lib.NNP_BUF_NBR_ANG, 1)):
        rows = m.read(which)
        out.append(np.where(np.arange(rows.shape[1])[None] < out[1][:, col:col + 1], rows, -1))
    out.append(m.read(P._lib.NNP_BUF_DESCRIPTOR))
    m.close()
    return ran, out


CASES = ["three_cells", "three_cells_tight", "flat", "moved", "far", "on_cutoff", "four_elements", "missing_species",
         "dense"]


@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("name", CASES)
def test_equal_lists(P, name, variant):
    pos, Z, box, cfg = inputs(name)
    caps = (512, 256) if name == "dense" else (256, 96)
    ran, ref = lists(P, cfg, pos, Z, box, 0, caps)
    assert ran == 0 and ref[0] == 0
    ran, got = lists(P, cfg, pos, Z, box, variant, caps)
    assert ran == (0 if name == "three_cells_tight" else variant)
    for a, b in zip(ref, got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("caps", [(40, 64), (128, 12), (59, 18), (17, 5)])
def test_equal_overflow(P, caps):
    """Lists cut at the same entries, and the status set."""
    pos, Z, box = sy.water_box(343, 21.74, seed=5)
    _, ref = lists(P, WATER, pos, Z, box, 0, caps)
    _, got = lists(P, WATER, pos, Z, box, 2, caps)
    assert ref[0] == P._lib.NNP_ECAPACITY
    for a, b in zip(ref, got):
        assert np.array_equal(a, b)
