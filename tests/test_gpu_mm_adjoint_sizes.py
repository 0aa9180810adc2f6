"""The MM-channel adjoint at the edges of its split: 8 NNP atoms per wavefront, up to 16
wavefronts per workgroup, 64 MM atoms per pass, workgroups that loop over MM atoms or over NNP
atoms, grid rows that add with atomics; MM forces overwritten or accumulated."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


def mm_lattice(pos, n_mm, rng):
    """n_mm sites of a 2.2 A lattice around the molecule, none within 2 A of an atom."""
    side = int(np.ceil((n_mm + 4 * len(pos)) ** (1 / 3))) + 2
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)
    g = (g - side / 2) * 2.2 + pos.mean(0)
    g = g[np.argsort(((g - pos.mean(0)) ** 2).sum(1))]
    d = np.min([((g - p) ** 2).sum(1) for p in pos], axis=0)
    return rng.permutation(g[d > 4.0][:n_mm]).astype(np.float32)


# FP32 pair terms and dE/dphi, FP64 sums: the FP32 form's 1e-5 of the forces
@pytest.mark.parametrize("n,n_mm", [(1, 1), (8, 63), (17, 129), (60, 3000), (128, 500), (129, 300), (200, 66000)])
def test_sizes(n, n_mm):
    import paper_2604_21441_amd as P
    cfg = sy.model_config("hcno_mm")
    rng = np.random.default_rng(n)
    pos, Z = sy.walk_molecule(max(n, 2), rng)
    pos, Z = pos[:n], Z[:n]
    mm = mm_lattice(pos.astype(np.float64), n_mm, rng)
    q = rng.uniform(-0.8, 0.8, n_mm).astype(np.float32)
    w = sy.model_weights(cfg, seed=2)
    m = P.NNPModel(cfg, weights=sy.flat_weights(w))
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = (torch.full((1,), 7.0, dtype=torch.float64, device="cuda"),
           torch.full((n, 3), 7.0, dtype=torch.float64, device="cuda"),
           torch.full((n_mm, 3), 7.0, dtype=torch.float64, device="cuda"))
    m.set_graph(True)
    for _ in range(2):   # the second call runs from the captured graph
        m.compute(t(pos), Z, None, None, t(mm), t(q), out=out)
    torch.cuda.synchronize()
    assert m.status() == 0
    E, F, Fmm = (a.cpu().numpy() for a in out)
    ref = orc.evaluate(pos, Z, cfg, w, mm_pos=mm, mm_q=q)
    assert abs(E[0] - ref["E"]) / n < 1e-6 * max(1.0, abs(ref["E"]) / n)
    assert np.linalg.norm(F - ref["F"]) < 1e-5 * np.linalg.norm(ref["F"])
    assert np.linalg.norm(Fmm - ref["F_mm"]) < 1e-5 * np.linalg.norm(ref["F_mm"])
    P.nnp_compute(m.h, t(pos), None, None, None, t(mm), t(q), out[0], out[1], out[2], accumulate=True)
    torch.cuda.synchronize()
    for a, b in zip(out, (E, F, Fmm)):
        assert np.allclose(a.cpu().numpy(), 2 * b, rtol=1e-12, atol=1e-12 * np.abs(b).max())
    m.close()
