"""nnp_compute_noalloc at its documented atom limits: the last size runs, one atom more is refused with
a message that names the limit."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,limit", [("water", 8960), ("hcno", 5752)])
def test_limit(kind, limit):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    rng = np.random.default_rng(1)
    side = int(np.ceil((limit + 1) ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)[:limit + 1] * 2.2
    pos = (g + rng.uniform(-0.2, 0.2, g.shape)).astype(np.float32)
    Z = rng.choice(np.array(cfg["species"], np.int32), limit + 1)
    box = np.full(3, 2.2 * side, np.float32)
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=1)))
    d = torch.from_numpy(pos).cuda()
    E = torch.zeros(1, dtype=torch.float64, device="cuda")
    F = torch.zeros((limit + 1, 3), dtype=torch.float64, device="cuda")
    with pytest.raises(P.NNPError) as ex:
        P.nnp_compute_noalloc(m.h, d, Z, box, E, F)
    assert ex.value.status == P._lib.NNP_ECAPACITY and str(limit) in str(ex.value) and "byte" not in str(ex.value)
    assert not F.any()
    P.nnp_compute_noalloc(m.h, d[:limit], Z[:limit], box, E, F[:limit])
    E0, F0, _ = m.compute(d[:limit], Z[:limit], box)
    torch.cuda.synchronize()
    assert m.status() == 0
    # the same kernels: the energy is a fixed-order FP64 sum, the forces differ by the order of FP64 additions
    assert E.item() == E0.item()
    assert torch.allclose(F[:limit], F0, rtol=0, atol=1e-10 * F0.abs().max().item())
    m.close()
