"""How calls are launched: a captured graph for few atoms, direct launches from three atoms per CU
on and with MM atoms, either one on request, all with the same results."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,per_cu,graph", [("water", -1, True), ("water", 2, True), ("water", 3, False),
                                               ("hcno_mm", -1, False)])
def test_launches(kind, per_cu, graph):
    import paper_2604_21441_amd as P
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    cfg = sy.model_config(kind)
    box = mm = q = None
    if kind == "water":
        n_mol = 64 if per_cu < 0 else (per_cu * n_cu) // 3 + 1
        pos, Z, box = sy.water_box(n_mol, 12.42 * (n_mol / 64) ** (1 / 3), seed=3)
    else:
        pos, Z = sy.walk_molecule(30, np.random.default_rng(4))
        mm = torch.from_numpy((pos + np.float32([0.0, 0.0, 8.0])).astype(np.float32)).cuda()
        q = torch.linspace(-0.5, 0.5, len(Z), device="cuda")
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=1)))
    x = torch.from_numpy(pos).cuda()
    counts, results = [], []
    for mode in (None, True, False):
        if mode is not None:
            m.set_graph(mode)
        out = (torch.zeros(1, dtype=torch.float64, device="cuda"), torch.zeros_like(x, dtype=torch.float64),
               None if mm is None else torch.zeros_like(mm, dtype=torch.float64))
        before = m.read(P._lib.NNP_BUF_GRAPH).sum() if results else 0
        for k in range(3):
            m.compute(x, Z if not results and k == 0 else None, box, None, mm, q, out=out)
            junk = torch.randn(2048, device="cuda").sum().item()   # unrelated eager work between calls
        torch.cuda.synchronize()
        assert m.status() == 0
        counts.append(int(m.read(P._lib.NNP_BUF_GRAPH).sum() - before))
        results.append([None if t is None else t.cpu() for t in out])
    assert counts == [3 if graph else 0, 3, 0]
    for r in results[1:]:
        for a, b in zip(results[0], r):
            assert a is None or torch.allclose(a, b, rtol=1e-12, atol=1e-12)
    m.close()
