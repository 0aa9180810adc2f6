"""The mechanical-embedding coupling at the edges of its split: ML atoms shared by 16
wavefronts and staged 256 at a time, MM atoms 128 to a workgroup in two tiles of 64."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


# FP32 pair terms summed in FP64 over a wavefront's partial sums in FP32: 1e-6 of the summed
# magnitudes for the energy, 1e-5 (rms) for the forces, as for the 60 x 30,000 workload
@pytest.mark.parametrize("n_ml,n_mm,periodic", [(1, 1, False), (7, 63, False), (16, 64, True), (17, 65, False), (3, 127, False), (10, 129, True),
                                                (256, 130, True), (257, 1000, False), (0, 5, False), (5, 0, False)])
def test_sizes(n_ml, n_mm, periodic):
    import paper_2604_21441_amd as P
    rng = np.random.default_rng(n_ml + 1000 * n_mm)
    side = int(np.ceil((n_ml + n_mm) ** (1 / 3)))
    g = rng.permutation(np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3))
    pos = (3.0 * g[:n_ml + n_mm] + rng.uniform(-0.3, 0.3, (n_ml + n_mm, 3))).astype(np.float32)
    par = np.stack([rng.uniform(-0.8, 0.8, n_ml + n_mm), rng.uniform(2.0, 3.3, n_ml + n_mm),
                    rng.uniform(0.001, 0.01, n_ml + n_mm)], 1).astype(np.float32)
    box = np.full(3, 3.0 * side, np.float32) if periodic else None
    cutoff = 1.4 * side if periodic else 0.0
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    x, q = (pos[:n_ml], pos[n_ml:]), (par[:n_ml], par[n_ml:])
    E, Fml, Fmm = P.nnp_me_coupling(t(x[0]), t(q[0]), t(x[1]), t(q[1]), box=box, cutoff=cutoff, ke=sy.KE_COULOMB)
    torch.cuda.synchronize()
    if n_ml == 0 or n_mm == 0:
        assert E.item() == 0.0 and not Fml.any() and not Fmm.any()
        return
    Er, Fml_r, Fmm_r, Eabs = orc.me_coupling(x[0], q[0], x[1], q[1], sy.KE_COULOMB, box=box,
                                             cutoff=cutoff if periodic else None, return_abs=True)
    assert abs(E.item() - Er) <= 1e-6 * Eabs
    F, R = np.concatenate([Fml.cpu().numpy(), Fmm.cpu().numpy()]), np.concatenate([Fml_r, Fmm_r])
    assert np.linalg.norm(F - R) <= 1e-5 * np.linalg.norm(R)
