"""The default neighbour kernel by what the box holds: cells for boxes filled at the density of
matter, one wavefront per atom for drops and gases in large boxes, cells much larger than the cutoff
and very long boxes; list lengths and forces are those of the pinned kernel."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu


def lattice(sides, spacing, species, rng):
    g = np.stack(np.meshgrid(*[np.arange(k) for k in sides], indexing="ij"), -1).reshape(-1, 3) * spacing
    return (g + rng.uniform(-0.15, 0.15, g.shape)).astype(np.float32), rng.choice(np.array(species, np.int32), len(g))


@pytest.mark.parametrize("kind,sides,spacing,box,cells", [
    ("water", (35, 35, 35), 2.15, (75.25, 75.25, 75.25), True),
    ("hcno", (35, 35, 35), 2.15, (75.25, 75.25, 75.25), True),
    ("water", (34, 34, 34), 2.15, (73.1, 73.1, 73.1), False),      # 39,304 atoms
    ("water", (36, 36, 36), 2.15, (300.0, 300.0, 300.0), False),   # a drop
    ("water", (36, 36, 36), 2.15, (77.4, 77.4, 154.8), False),     # a slab
    ("water", (37, 37, 37), 6.0, (222.0, 222.0, 222.0), False),    # a gas
    ("water", (9, 9, 520), 2.3, (20.7, 20.7, 1196.0), False),      # long, cells of 6.9 A
    ("hcno", (40, 40, 40), 1.95, (78.0, 78.0, 78.0), True),
    ("hcno", (35, 35, 35), 1.95, (68.25, 68.25, 68.25), False),    # 42,875 atoms
])
def test_choice(kind, sides, spacing, box, cells):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    pos, Z = lattice(sides, spacing, (1, 1, 8) if kind == "water" else (1, 6, 7, 8), np.random.default_rng(3))
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=1)))
    m.reserve(len(Z), max_rad_nbr=160, max_ang_nbr=96)
    d, box = torch.from_numpy(pos).cuda(), np.array(box, np.float32)
    counts = []
    for pin in (-1, 0):
        m.set_variant("neighbours", pin)
        E, F, _ = m.compute(d, Z, box)
        torch.cuda.synchronize()
        assert m.status() == 0
        if pin < 0:
            assert (m.variants()["neighbours"] > 0) == cells
        counts.append((m.read(P._lib.NNP_BUF_NBR_COUNT).copy(), F.cpu().numpy()))
    assert np.array_equal(counts[0][0], counts[1][0])
    assert np.allclose(counts[0][1], counts[1][1], rtol=0, atol=1e-9 * np.abs(counts[1][1]).max())
    m.close()
