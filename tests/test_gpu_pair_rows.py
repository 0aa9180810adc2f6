"""Lists from a caller's pair list at the edges of the row sort: rows of one to four entries
per lane, up to the largest capacity, capacities that cut rows off, and pairs given twice."""
import numpy as np
import pytest
import torch

import oracle as orc
import synthetic as sy

pytestmark = pytest.mark.gpu

HCNO = sy.model_config("hcno")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    import paper_2604_21441_amd as P
    return P


def cluster(spacing, side=9):
    rng = np.random.default_rng(5)
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3) * spacing
    pos = (g + rng.uniform(-0.08, 0.08, g.shape)).astype(np.float32)
    Z = rng.choice(np.array([1, 6, 7, 8], dtype=np.int32), size=len(pos))
    I, J = orc.neighbour_pairs(pos, 5.6, None)
    pairs = np.stack([I[I < J], J[I < J]], 1).astype(np.int32)
    return pos, Z, pairs[rng.permutation(len(pairs))]


def lists(P, m):
    cnt = m.read(P._lib.NNP_BUF_NBR_COUNT)
    out = [cnt]
    for buf, col in ((P._lib.NNP_BUF_NBR_RAD, 0), (P._lib.NNP_BUF_NBR_ANG, 1)):
        r = m.read(buf)
        out.append(np.where(np.arange(r.shape[1])[None, :] < cnt[:, col:col + 1], r, -1))
    return out


@pytest.mark.parametrize("spacing,max_rad,max_ang", [(4.0, 128, 64), (2.0, 127, 64), (1.5, 255, 64), (1.36, 256, 128)])
def test_rows_match_the_search(P, spacing, max_rad, max_ang):
    """The same lists, energy and forces, bit for bit, as from the library's own search."""
    pos, Z, pairs = cluster(spacing)
    w = sy.flat_weights(sy.model_weights(HCNO, seed=1))
    d = torch.from_numpy(pos).cuda()
    got = []
    for listed in (False, True):
        m = P.NNPModel(HCNO, weights=w)
        m.reserve(len(Z), 1, 0, max_rad, max_ang)
        E, F, _ = m.compute_pairs(d, torch.from_numpy(pairs).cuda(), Z) if listed else m.compute(d, Z)
        torch.cuda.synchronize()
        assert m.status() == 0
        got.append(lists(P, m) + [E.cpu().numpy(), F.cpu().numpy()])
        m.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    lo, hi = {4.0: (1, 20), 2.0: (65, 128), 1.5: (129, 192), 1.36: (193, 256)}[spacing]
    assert lo <= got[0][0][:, 0].max() <= hi   # entries per lane: 1, 2, 3, 4


def test_pair_given_twice_and_cut_rows(P):
    """A repeated pair is an input error, and its row lists it twice, in order; rows beyond the
    capacity are cut off and flagged."""
    pos, Z, pairs = cluster(1.5)
    w = sy.flat_weights(sy.model_weights(HCNO, seed=1))
    d = torch.from_numpy(pos).cuda()
    m = P.NNPModel(HCNO, weights=w)
    m.reserve(len(Z), 1, 0, 256, 128)
    r = np.linalg.norm(pos[pairs[:, 0]] - pos[pairs[:, 1]], axis=1)
    again = pairs[np.argmin(r)]
    m.compute_pairs(d, torch.from_numpy(np.concatenate([pairs, again[None]])).cuda(), Z)
    torch.cuda.synchronize()
    assert m.status() == P._lib.NNP_EINVAL
    perm = m.read(P._lib.NNP_BUF_PERM)
    cnt, rad, ang = lists(P, m)
    for a, b in (again, again[::-1]):
        i, j = np.nonzero(perm == a)[0][0], np.nonzero(perm == b)[0][0]
        row = rad[i, :cnt[i, 0]]
        assert np.all(np.diff(row) >= 0) and np.sum(row == j) == 2 and len(set(row)) == len(row) - 1
    m.reserve(len(Z), 1, 0, 100, 30)
    m.compute_pairs(d, torch.from_numpy(pairs).cuda(), Z)
    torch.cuda.synchronize()
    assert m.status() == P._lib.NNP_ECAPACITY
    cnt, rad, ang = lists(P, m)
    assert cnt[:, 0].max() == 100
    assert all(np.all(np.diff(rad[i, :c]) > 0) for i, c in enumerate(cnt[:, 0]))
    m.close()
