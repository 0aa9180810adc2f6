"""The MM channel with larger ML regions: the adjoint's four MM atoms per lane, grid rows and
several passes over the MM atoms, and the workspace that nnp_reserve takes for it."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


def region(n, n_mm, rng):
    """n atoms on a jittered 2 A lattice inside a shuffled 2.2 A lattice of n_mm charges."""
    k = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * 2.0
    pos = (g + rng.uniform(-0.1, 0.1, g.shape)).astype(np.float32)
    km = int(np.ceil((n_mm + 8 * n + 64) ** (1 / 3))) + 2
    gm = (np.stack(np.meshgrid(*[np.arange(km)] * 3, indexing="ij"), -1).reshape(-1, 3) - km / 2) * 2.2 + k
    gm = gm[((gm < -1.5) | (gm > 2.0 * k - 0.5)).any(1)]
    gm = gm[np.argsort(((gm - k) ** 2).sum(1))][:n_mm]
    assert len(gm) == n_mm
    return pos, rng.choice(np.array([1, 6, 7, 8], np.int32), n), rng.permutation(gm).astype(np.float32)


# FP32 pair terms and dE/dphi, sums over 64 lanes and up to 32 pairs per lane in FP32, the rest FP64:
# the FP32 form's 1e-5 of the forces
@pytest.mark.parametrize("n,n_mm,graph", [(1, 40000, False), (9, 33000, True), (99, 30001, False), (137, 29999, True),
                                          (520, 4100, True), (1025, 3000, False), (40, 140000, False)])
@pytest.mark.parametrize("kind", ["hcno_mm", "hcno_ee"])
def test_sizes(kind, n, n_mm, graph):
    import paper_2604_21441_amd as P
    cfg = sy.model_config(kind)
    rng = np.random.default_rng(n)
    pos, Z, mm = region(n, n_mm, rng)
    q = rng.uniform(-0.8, 0.8, n_mm).astype(np.float32)
    w = sy.model_weights(cfg, seed=2)
    m = P.NNPModel(cfg, weights=sy.flat_weights(w))
    m.set_graph(graph)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    x, y, c = t(pos), t(mm), t(q)
    out = tuple(torch.full(s, 7.0, dtype=torch.float64, device="cuda") for s in ((1,), (n, 3), (n_mm, 3)))
    for _ in range(3):
        m.compute(x, Z, None, None, y, c, out=out)
    torch.cuda.synchronize()
    assert m.status() == 0
    E, F, Fmm = (a.cpu().numpy() for a in out)
    near = np.flatnonzero((((mm[:, None, :] - pos[None, ::7]) ** 2).sum(-1) < 30.0 ** 2).any(1))   # (the others have no part)
    ref = orc.evaluate(pos, Z, cfg, w, mm_pos=mm[near], mm_q=q[near])
    assert abs(E[0] - ref["E"]) / n < 1e-6 * max(1.0, abs(ref["E"]) / n)
    assert np.linalg.norm(F - ref["F"]) < 1e-5 * np.linalg.norm(ref["F"])
    assert np.linalg.norm(Fmm[near] - ref["F_mm"]) < 1e-5 * np.linalg.norm(ref["F_mm"])
    Fmm[near] = 0.0
    assert not Fmm.any()
    P.nnp_compute(m.h, x, None, None, None, y, c, out[0], out[1], out[2], accumulate=True)
    torch.cuda.synchronize()
    Fmm = out[2].cpu().numpy()
    assert np.allclose(out[1].cpu().numpy(), 2 * F, rtol=1e-12, atol=1e-12 * np.abs(F).max())
    assert np.linalg.norm(Fmm[near] - 2 * ref["F_mm"]) < 2e-5 * np.linalg.norm(ref["F_mm"])
    m.close()


@pytest.mark.parametrize("atoms,charges", [(100000, 30000), (60, 30000), (30060, 30000), (100, 100)])
def test_reserved_memory(atoms, charges):
    """12 bytes per atom and 256 charges, or up to four times that within 1,536 bytes per CU."""
    import paper_2604_21441_amd as P
    cfg = sy.model_config("hcno_mm")
    m = P.NNPModel(cfg, weights=sy.flat_weights(sy.model_weights(cfg, seed=1)))
    torch.cuda.synchronize()
    used = []
    for mm in (0, charges):
        m.reserve(atoms, 1, mm)
        used.append(-torch.cuda.mem_get_info()[0])
    groups = -(-charges // 256)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    most = max(12 * atoms * groups, min(4 * 12 * atoms * groups, 1536 * cus))
    assert used[1] - used[0] <= most + (4 << 20)   # (allocations come in pages of up to 2 MiB)
    m.close()
