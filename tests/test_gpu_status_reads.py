"""The status word is read and cleared by the caller at any time, on any stream: neither a word
left from an earlier call nor one cleared while a call runs changes that call's forces."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

WATER = sy.model_config("water")


def test_cleared_while_a_call_runs():
    """Lists cut off at their capacity (the contributions then follow the radial lists), the status
    read on another stream at moments spread over the call."""
    import paper_2604_21441_amd as P
    pos, Z, box = sy.water_box(4096, 12.42 * 4, seed=5)
    m = P.NNPModel(WATER, weights=sy.flat_weights(sy.model_weights(WATER, seed=1)))
    m.reserve(len(Z), max_rad_nbr=45, max_ang_nbr=20)
    x = torch.from_numpy(pos).cuda()
    call, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    out = (torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty_like(x, dtype=torch.float64), None)
    m.compute(x, Z, box, out=out, stream=call)
    torch.cuda.synchronize()
    assert m.status() == P._lib.NNP_ECAPACITY
    ref = out[1].cpu().numpy()
    for _ in range(40):
        m.compute(x, None, box, out=out, stream=call)
        seen = 0
        while not call.query():
            seen = seen or m.status(stream=other)
        torch.cuda.synchronize()
        assert P._lib.NNP_ECAPACITY in (seen, m.status())
        F = out[1].cpu().numpy()
        assert np.abs(F - ref).max() < 1e-10 * np.abs(ref).max()
    m.close()


def test_left_from_an_earlier_call():
    import paper_2604_21441_amd as P
    w = sy.model_weights(WATER, seed=1)
    big, ZB, boxB = sy.water_box(343, 21.74, seed=5)
    pos, Z, _ = sy.water_box(8, 8.0, seed=3)   # a drop, whose lists fit
    m = P.NNPModel(WATER, weights=sy.flat_weights(w))
    m.reserve(len(ZB), max_rad_nbr=32, max_ang_nbr=16)
    m.compute(torch.from_numpy(big).cuda(), ZB, boxB)
    E, F, _ = m.compute(torch.from_numpy(pos).cuda(), Z)
    torch.cuda.synchronize()
    assert m.status() == P._lib.NNP_ECAPACITY   # (the first call's)
    ref = orc.evaluate(pos, Z, WATER, w)
    assert abs(E.item() - ref["E"]) < 1e-6 * len(Z)
    assert np.linalg.norm(F.cpu().numpy() - ref["F"]) < 1e-5 * np.linalg.norm(ref["F"])
    m.close()
