"""Sparse chains whose rows have at most 16 entries run four steps at a time.  Rows that share columns (inside a
group of four, and at every distance the early fetches reach over), rows that are empty, full or longer, and chains that
end inside a group, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (groups of four from 128 steps on; the others run one step at a time)
STEPS = np.array([0, 1, 3, 4, 5, 31, 32, 33, 64, 127, 128, 129, 130, 131, 159, 160, 161, 191, 193, 255, 514, 700], dtype=np.int64)
# fp64 state leaves the rounding of the result (6e-8 an element); fp32 state some 700 roundings of it
TOL = {wl.HINGE: 2e-7, wl.LOGISTIC: 2e-5}


def _matrix(rng, m, d, lens, hot):
    """Rows of the given lengths; a share `hot` of the entries falls on forty columns spread over the range."""
    spots = np.unique(np.linspace(0, d - 1, 40).astype(np.int64))
    cols, vals, ptr = [], [], [0]
    for ln in lens:
        c = np.where(rng.random(ln * 3 + 8) < hot, rng.choice(spots, ln * 3 + 8), rng.integers(0, d, ln * 3 + 8))
        c = np.unique(c)
        c = np.sort(rng.permutation(c)[:ln])
        v = rng.standard_normal(c.size).astype(np.float32)
        cols.append(c.astype(np.int32))
        vals.append(v / max(np.linalg.norm(v), 1e-6))
        ptr.append(ptr[-1] + c.size)
    return np.array(ptr, dtype=np.int64), np.concatenate(cols), np.concatenate(vals).astype(np.float32)


def _run(ptr, cols, vals, m, d, loss, seed, **kw):
    rng = np.random.default_rng(seed)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    X = api.Matrix(m, d, row_ptr=torch.from_numpy(ptr).cuda(), col_idx=torch.from_numpy(cols).cuda(), vals=torch.from_numpy(vals).cuda())
    yg = torch.from_numpy(y).cuda()
    W = api.wpsgd_run_chains(X, yg, STEPS, 0.4, 1e-3, loss, 7, **kw)
    ref = orc.run_chains(orc.CSR(ptr, cols, vals, d), y, STEPS, 0.4, 1e-3, loss, 7)[0]
    got = W.cpu().numpy()
    for i in range(len(STEPS)):
        assert np.linalg.norm(got[i] - ref[i]) <= TOL[loss] * max(np.linalg.norm(ref[i]), 1e-30), i
    assert torch.equal(W, api.wpsgd_run_chains(X, yg, STEPS, 0.4, 1e-3, loss, 7, **kw))


@pytest.mark.parametrize("d", [128, 200, 8191, 8193, 30000])
@pytest.mark.parametrize("hot", [0.0, 0.1, 0.6])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_rows_that_share_columns(d, hot, loss):
    rng = np.random.default_rng(d + int(10 * hot))
    m = 900
    _run(*_matrix(rng, m, d, rng.integers(0, 17, size=m), hot), m, d, loss, d)


@pytest.mark.parametrize("d", [300, 30000])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_a_few_long_rows_among_short_ones(d, loss):
    rng = np.random.default_rng(d)
    m = 3000                                       # every fourth row or so is looked at; the long ones lie between
    lens = rng.integers(0, 17, size=m)
    looked = {i * m // 768 for i in range(768)}
    free = [j for j in range(m) if j not in looked]
    for q, j in enumerate(rng.choice(free, 400, replace=False)):
        lens[j] = [17, 40, 64, 65, 130][q % 5]
    _run(*_matrix(rng, m, d, lens, 0.2), m, d, loss, d)


def test_all_rows_empty_but_one():
    ptr = np.zeros(101, dtype=np.int64)
    ptr[51:] = 3
    _run(ptr, np.array([1, 9000, 9001], dtype=np.int32), np.array([0.5, 0.5, 0.7], dtype=np.float32), 100, 9100, wl.HINGE, 3)
