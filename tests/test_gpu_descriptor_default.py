"""The default descriptor kernel on both sides of the sizes where it changes: one and two
atoms per wavefront of the pool kernel (eight atoms per CU), and for two elements the pool,
the row kernel and the pool again (24 and 72 atoms per CU)."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

HCNO = sy.model_config("hcno")
WATER = sy.model_config("water")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    import paper_2604_21441_amd as P
    return P


def n_cu():
    return torch.cuda.get_device_properties(0).multi_processor_count


# FP32 sums of some hundred terms of one sign: 5e-6 of a row's norm,
# as for the kernels when pinned
@pytest.mark.parametrize("extra", [-2047, 0, 1])
def test_hcno_pool_split(P, extra):
    n = max(1, 8 * n_cu() + extra)
    pos, Z, off = sy.walk_batch(64, seed=21)
    assert len(Z) > n
    off = np.append(off[off < n], n)
    w = sy.model_weights(HCNO, seed=1)
    m = P.NNPModel(HCNO, weights=sy.flat_weights(w))
    E, F = m.compute_batch(torch.from_numpy(pos[:n]).cuda(), Z[:n], off)
    torch.cuda.synchronize()
    assert m.status() == 0 and m.variants()["descriptor"] == 3
    x = np.empty((n, 384), dtype=np.float32)
    x[m.read(P._lib.NNP_BUF_PERM)] = m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :384]
    for s in sorted({0, (len(off) - 1) // 2, len(off) - 2}):
        a, b = off[s], off[s + 1]
        ref = orc.evaluate(pos[a:b], Z[a:b], HCNO, w, return_x=True)["x"]
        err = np.linalg.norm(x[a:b] - ref, axis=1)
        assert np.all(err <= 5e-6 * np.linalg.norm(ref, axis=1)), (s, err.max())
    m.close()


@pytest.mark.parametrize("per_cu,below,above", [(24, 3, 1), (72, 1, 4)])
def test_water_sizes(P, per_cu, below, above):
    w = sy.flat_weights(sy.model_weights(WATER, seed=1))
    for n_mol, variant in (((per_cu * n_cu() - 1) // 3, below), (per_cu * n_cu() // 3 + 1, above)):
        pos, Z, box = sy.water_box(n_mol, 12.42 * (n_mol / 64) ** (1 / 3), seed=3)
        d = torch.from_numpy(pos).cuda()
        m = P.NNPModel(WATER, weights=w)
        rows = []
        for pin in (-1, 0):   # the default, and one wavefront per atom
            m.set_variant("descriptor", pin)
            m.compute(d, Z, box)
            torch.cuda.synchronize()
            assert m.status() == 0
            if pin < 0:
                assert m.variants()["descriptor"] == variant
            rows.append(m.read(P._lib.NNP_BUF_DESCRIPTOR)[:, :128].copy())
        err = np.linalg.norm(rows[0] - rows[1], axis=1)
        assert np.all(err <= 5e-6 * np.linalg.norm(rows[1], axis=1)), err.max()
        m.close()
