"""Sparse chains whose short rows hardly ever share a column run sixteen steps at a time, and what a value requested early lacks is
added from the rows alone.  Columns that come back at every distance, rows of every length, chains that end anywhere in a block,
elements that are not finite, against the oracle or the one-wave kernel."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

M, D, SEED = 4096, 300000, 17
# (sixteen steps at a time from 128 steps on; the others run one at a time)
STEPS = np.array([700, 127, 128, 129, 143, 144, 145, 160, 191, 193, 207, 208, 209, 255, 0, 1], dtype=np.int64)
# fp64 state leaves the rounding of the result (6e-8 an element); fp32 state some 700 roundings of it
TOL = {wl.HINGE: 2e-7, wl.LOGISTIC: 2e-5}
APART = 3                                      # what the look at the matrix leaves in the word behind the status word
LOOKED = {i * M // 768 for i in range(768)}    # rows it may have looked at: no column is planted there


def _rows(rng, planted, lens=None):
    ptr, cols, vals = [0], [], []
    for r in range(M):
        ln = 8 if lens is None else int(lens[r])
        own = rng.integers(0, D - 4096, size=ln)
        keep = planted.get(r, []) if r not in LOOKED else []
        c = np.unique(np.concatenate([own[:max(0, ln - len(keep))], np.array(keep, dtype=np.int64) + D - 4096]).astype(np.int64))
        v = rng.standard_normal(c.size).astype(np.float32)
        cols.append(c.astype(np.int32))
        vals.append(v / max(np.linalg.norm(v), 1e-6))
        ptr.append(ptr[-1] + c.size)
    return np.array(ptr, dtype=np.int64), np.concatenate(cols), np.concatenate(vals).astype(np.float32)


def _first_visits(n):
    first = {}
    for t, r in enumerate(api.wpsgd_sample_indices(SEED, 0, 0, n, M).tolist()):
        first.setdefault(r, t)
    return first


def _run(ptr, cols, vals, loss, **kw):
    y = np.where(np.random.default_rng(1).random(M) < 0.5, 1.0, -1.0).astype(np.float32)
    X = api.Matrix(M, D, row_ptr=torch.from_numpy(ptr).cuda(), col_idx=torch.from_numpy(cols).cuda(), vals=torch.from_numpy(vals).cuda())
    ws = torch.empty(api.wpsgd_run_chains_workspace(X, len(STEPS), loss), dtype=torch.uint8, device="cuda")
    yg = torch.from_numpy(y).cuda()
    W = api.wpsgd_run_chains_from(X, yg, STEPS, 0.4, 1e-3, loss, SEED, workspace=ws, **kw)
    assert int(ws[4:8].view(torch.int32).item()) == APART
    assert torch.equal(torch.nan_to_num(W, 7.0), torch.nan_to_num(api.wpsgd_run_chains_from(X, yg, STEPS, 0.4, 1e-3, loss, SEED, workspace=ws, **kw), 7.0))
    return X, yg, y, W


def _check(ptr, cols, vals, loss):
    _, _, y, W = _run(ptr, cols, vals, loss)
    ref = orc.run_chains(orc.CSR(ptr, cols, vals, D), y, STEPS, 0.4, 1e-3, loss, SEED)[0]
    got = W.cpu().numpy()
    for i in range(len(STEPS)):
        assert np.linalg.norm(got[i] - ref[i]) <= TOL[loss] * max(np.linalg.norm(ref[i]), 1e-30), i


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("period", [1, 2, 3, 4, 5, 8, 12, 15, 16, 17, 24, 31, 32, 33, 47, 64])
def test_columns_that_come_back(period, loss):
    """Rows first visited `period` steps apart share three columns: within four rows taken side by side, within a block, with the block
    before, and just further back, where the early request must already see the last write.  Small periods have more pairs than the lists hold."""
    planted = {r: [3 * (t % period) + q for q in range(3)] for r, t in _first_visits(700).items()}
    _check(*_rows(np.random.default_rng(period), planted), loss)


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("share", [2, 3, 9])
def test_some_rows_in_a_row_share_columns(share, loss):
    """`share` steps out of every forty share two columns, so that pairs follow from pairs."""
    planted = {r: [2 * (t // 40) % 500, 2 * (t // 40) % 500 + 1] for r, t in _first_visits(700).items() if t % 40 < share}
    _check(*_rows(np.random.default_rng(share), planted), loss)


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_rows_of_every_length_and_a_few_long_ones(loss):
    rng = np.random.default_rng(5)
    lens = rng.integers(0, 17, size=M)
    free = [r for r in range(M) if r not in LOOKED]
    for q, r in enumerate(rng.choice(free, 150, replace=False)):
        lens[r] = [17, 40, 64, 65, 130][q % 5]
    planted = {r: [t % 20] for r, t in _first_visits(700).items() if lens[r] > 2}
    _check(*_rows(rng, planted, lens), loss)


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_start_vector_and_shares_of_the_rows(loss):
    ptr, cols, vals = _rows(np.random.default_rng(6), {})
    start = torch.from_numpy(np.random.default_rng(7).standard_normal(D).astype(np.float32) * 0.1).cuda()
    for kw in ({"w_start": start}, {"sampling": api.SAMPLE_SHARDS}, {"w_start": start, "sampling": api.SAMPLE_SHARDS}):
        X, yg, _, W = _run(ptr, cols, vals, loss, **kw)
        other = api.wpsgd_run_chains_from(X, yg, STEPS, 0.4, 1e-3, loss, SEED, plan={"prefetch": 4}, **kw)
        for i in range(len(STEPS)):
            assert (W[i] - other[i]).double().norm() <= TOL[loss] * max(other[i].double().norm().item(), 1e-30), i


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_elements_that_are_not_finite(bad, loss):
    first = _first_visits(700)
    ptr, cols, vals = _rows(np.random.default_rng(8), {r: [t % 30] for r, t in first.items()})
    row = next(r for r, t in first.items() if t == 300)
    vals[ptr[row] + 2] = bad
    X, yg, _, W = _run(ptr, cols, vals, loss)
    other = api.wpsgd_run_chains_from(X, yg, STEPS, 0.4, 1e-3, loss, SEED, plan={"prefetch": 4})
    assert torch.equal(torch.isfinite(W), torch.isfinite(other)) and not torch.isfinite(W[0]).all()
    W, other = torch.nan_to_num(W, 0.0, 0.0, 0.0), torch.nan_to_num(other, 0.0, 0.0, 0.0)
    for i in range(len(STEPS)):
        assert (W[i] - other[i]).double().norm() <= TOL[loss] * max(other[i].double().norm().item(), 1e-30), i
