"""The coupling around the size where a workgroup has 4 wavefronts instead of 16 (2,048 workgroups of
128 MM atoms), with MM atoms beyond the cutoff in most workgroups."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu


# FP32 pair terms summed in FP64 over a wavefront's partial sums in FP32: as for the smaller sizes
@pytest.mark.parametrize("n_mm", [262144, 262145, 300001])
@pytest.mark.parametrize("n_ml", [1, 5, 270])
def test_sizes(n_ml, n_mm):
    import paper_2604_21441_amd as P
    rng = np.random.default_rng(n_ml)
    k = int(np.ceil((n_ml + n_mm) ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n_ml + n_mm] * 3.0
    near = np.argsort(((g - 1.5 * k) ** 2).sum(1))
    pos = (g + rng.uniform(-0.3, 0.3, g.shape)).astype(np.float32)
    x, y = pos[near[:n_ml]], pos[np.sort(near[n_ml:])]
    par = [np.stack([rng.uniform(-0.8, 0.8, n), rng.uniform(2.0, 3.3, n), rng.uniform(0.001, 0.01, n)], 1)
           .astype(np.float32) for n in (n_ml, n_mm)]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    args = (t(x), t(par[0]), t(y), t(par[1]))
    out = P.nnp_me_coupling(*args, cutoff=12.0, ke=sy.KE_COULOMB)
    torch.cuda.synchronize()
    E, Fml, Fmm = (o.cpu().numpy().copy() for o in out)
    close = np.flatnonzero(((y - x.mean(0)) ** 2).sum(1) < 45.0 ** 2)   # (the others have no part)
    Er, Rml, Rmm, Eabs = orc.me_coupling(x, par[0], y[close], par[1][close], sy.KE_COULOMB, cutoff=12.0, return_abs=True)
    assert abs(E[0] - Er) <= 1e-6 * Eabs
    F, R = np.concatenate([Fml, Fmm[close]]), np.concatenate([Rml, Rmm])
    assert np.linalg.norm(F - R) <= 1e-5 * np.linalg.norm(R)
    Fmm[close] = 0.0
    assert not Fmm.any()
    P.nnp_me_coupling(*args, cutoff=12.0, ke=sy.KE_COULOMB, accumulate=True, out=out)
    torch.cuda.synchronize()
    assert np.allclose(out[1].cpu().numpy(), 2 * Fml, rtol=1e-9, atol=1e-9 * np.abs(Fml).max())
    assert np.allclose(out[2].cpu().numpy()[close], 2 * Rmm, rtol=0, atol=2e-5 * np.abs(Rmm).max())
