"""The cell neighbour kernel where cells hold more candidates than its registers (512 or 768) and its
list in LDS (512 more): the same lists, species segments and overflow status as one wavefront per
atom, bit for bit, in filled boxes and for a drop whose cells are much denser than the average."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu


def lattice(sides, spacing, species, seed=11):
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(k) for k in sides], indexing="ij"), -1).reshape(-1, 3) * spacing
    return (g + rng.uniform(-0.12, 0.12, g.shape)).astype(np.float32), rng.choice(np.array(species, np.int32), len(g))


def lists(P, cfg, pos, Z, box, variant, caps):
    m = P.NNPModel(cfg, seed=1)
    m.reserve(len(Z), max_rad_nbr=caps[0], max_ang_nbr=caps[1])
    m.set_variant("neighbours", variant)
    m.compute(torch.from_numpy(pos).cuda(), Z, box)
    torch.cuda.synchronize()
    assert m.variants()["neighbours"] == variant
    out = [m.status(), m.read(P._lib.NNP_BUF_NBR_COUNT)]
    for which, col in ((P._lib.NNP_BUF_NBR_RAD, 0), (P._lib.NNP_BUF_NBR_ANG, 1)):
        rows = m.read(which)
        out.append(np.where(np.arange(rows.shape[1])[None] < out[1][:, col:col + 1], rows, -1))
    out.append(m.read(P._lib.NNP_BUF_DESCRIPTOR))
    m.close()
    return out


@pytest.mark.parametrize("kind", ["water", "hcno"])
@pytest.mark.parametrize("spacing,box,caps", [
    (1.9, 24.7, (256, 96)),      # 13 x 13 x 13 in 4 x 4 x 4 cells: about 930 candidates
    (1.72, 22.36, (256, 128)),   # about 930, cells of 5.6 A
    (1.3, 22.1, (512, 256)),     # about 2,070: beyond the LDS list as well
    (2.1, 60.0, (256, 96)),      # a drop in a box five times its volume
    (1.72, 22.36, (90, 128)),    # cut off
    (1.3, 22.1, (512, 60)),
])
def test_equal_lists(kind, spacing, box, caps):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    side = int(round(min(box, 27.3) / spacing))
    pos, Z = lattice((side,) * 3, spacing, (1, 8) if kind == "water" else (1, 6, 7, 8))
    box = np.full(3, box, np.float32)
    ref = lists(P, cfg, pos, Z, box, 0, caps)
    assert (ref[0] != 0) == (caps in ((90, 128), (512, 60)))
    for variant in (1, 2, 3):
        for a, b in zip(ref, lists(P, cfg, pos, Z, box, variant, caps)):
            assert np.array_equal(a, b)


def test_missing_species_behind_the_registers():
    """One species fills the registers, the next starts behind them, two are missing."""
    import paper_2604_21441_amd as P
    cfg = sy.model_config("hcno")
    pos, Z = lattice((14,) * 3, 1.6, (6,))
    Z[::97] = 8
    box = np.full(3, 22.4, np.float32)
    ref = lists(P, cfg, pos, Z, box, 0, (256, 160))
    assert ref[0] == 0
    for variant in (1, 2, 3):
        for a, b in zip(ref, lists(P, cfg, pos, Z, box, variant, (256, 160))):
            assert np.array_equal(a, b)
