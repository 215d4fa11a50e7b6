"""The evaluator at the sizes where a row's lanes, a wave's 64 results or the copy of the model's head end."""
import math

import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _check(out, z, w, lam, loss):
    l = np.maximum(0.0, 1.0 - z) if loss == wl.HINGE else np.logaddexp(0.0, -z)
    want = 0.5 * lam * (w @ w) + l.mean()
    # fp64 sums of m terms in another order: at most m * 2^-53 relative, far below this
    assert abs(out[0] - want) <= 1e-10 * max(1.0, abs(want))
    assert abs(out[1] - (z <= 0).mean()) * z.size <= 1.0                   # one row may sit on zero


@pytest.mark.parametrize("d", [1, 3, 4, 5, 15, 16, 17, 31, 33, 63, 65, 127, 128, 129, 250, 513, 1100])
@pytest.mark.parametrize("m", [1, 63, 64, 65, 1000])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_dense_rows(d, m, bf16, loss):
    rng = np.random.default_rng(d * 1000 + m)
    X = rng.standard_normal((m, d)).astype(np.float32)
    dev = torch.from_numpy(X).cuda()
    if bf16:
        dev = dev.to(torch.bfloat16)
        X = dev.float().cpu().numpy()
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    w = (rng.standard_normal(d) / math.sqrt(d)).astype(np.float32)
    out = api.wpsgd_objective(api.Matrix(m, d, dense=dev), torch.from_numpy(y).cuda(), torch.from_numpy(w).cuda(), 0.01, loss).cpu().numpy()
    _check(out, y * (X.astype(np.float64) @ w.astype(np.float64)), w.astype(np.float64), 0.01, loss)


@pytest.mark.parametrize("m", [1, 3, 5, 1000, 40000, 131071, 131072, 140001])
@pytest.mark.parametrize("d", [7, 16384, 16385, 40000])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_sparse_rows(m, d, loss):
    rng = np.random.default_rng(m + d)
    lens = rng.integers(0, 8, size=m)
    lens[rng.integers(0, m, size=3)] = [0, 16, 300]
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cols = rng.integers(0, d, size=ptr[-1]).astype(np.int32)               # (the evaluator needs no order, nor distinct columns)
    vals = rng.standard_normal(ptr[-1]).astype(np.float32)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    w = rng.standard_normal(d).astype(np.float32)
    pad = lambda a: torch.from_numpy(a if a.size else np.zeros(1, a.dtype)).cuda()
    X = api.Matrix(m, d, row_ptr=pad(ptr), col_idx=pad(cols), vals=pad(vals))
    out = api.wpsgd_objective(X, torch.from_numpy(y).cuda(), torch.from_numpy(w).cuda(), 0.01, loss).cpu().numpy()
    z = y * np.bincount(np.repeat(np.arange(m), lens), weights=w.astype(np.float64)[cols] * vals.astype(np.float64), minlength=m)
    _check(out, z, w.astype(np.float64), 0.01, loss)


@pytest.mark.parametrize("d", [4, 5, 18, 31, 63, 99, 127])
def test_an_infinite_element_counts_once(d):
    """z = +inf costs nothing, z = -inf is wrong and costs infinitely much; no lane may meet the element with a weight of zero."""
    X = torch.ones((70, d), device="cuda")
    X[3, d - 1] = math.inf
    X[65, d - 1] = math.inf
    y = torch.ones(70, device="cuda")
    w = torch.full((d,), 0.25, device="cuda")
    out = api.wpsgd_objective(api.Matrix(70, d, dense=X), y, w, 0.0, wl.HINGE).cpu().numpy()
    assert abs(out[0] - max(0.0, 1.0 - 0.25 * d) * 68 / 70) < 1e-12
    assert out[1] == 0.0
    y[65] = -1.0
    out = api.wpsgd_objective(api.Matrix(70, d, dense=X), y, w, 0.0, wl.HINGE).cpu().numpy()
    assert out[0] == math.inf and abs(out[1] - 1.0 / 70) < 1e-15


def _sparse(lens, d):
    rng = np.random.default_rng(int(lens.size))
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cols = rng.integers(0, d, size=ptr[-1]).astype(np.int32)
    vals = rng.standard_normal(ptr[-1]).astype(np.float32)
    y = np.where(rng.random(lens.size) < 0.5, 1.0, -1.0).astype(np.float32)
    w = (rng.standard_normal(d) / 8).astype(np.float32)
    X = api.Matrix(lens.size, d, row_ptr=torch.from_numpy(ptr).cuda(), col_idx=torch.from_numpy(cols).cuda(), vals=torch.from_numpy(vals).cuda())
    z = y * np.bincount(np.repeat(np.arange(lens.size), lens), weights=w.astype(np.float64)[cols] * vals.astype(np.float64), minlength=lens.size)
    return X, torch.from_numpy(y).cuda(), torch.from_numpy(w).cuda(), z


def _best_us(X, y, w):
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    ws = torch.empty(max(256, api.wpsgd_objective_workspace(X)), dtype=torch.uint8, device="cuda")
    best = float("inf")
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            api.wpsgd_objective(X, y, w, 0.01, wl.HINGE, out=out, workspace=ws)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 200.0)
    return best, out.cpu().numpy()


@pytest.mark.parametrize("m", [5, 300, 5000, 20000, 150000, 420000])
@pytest.mark.parametrize("kind", ["one_long", "many_long", "all_long"])
def test_sparse_rows_longer_than_a_batch_takes(m, kind):
    """Rows of more than 256 entries go through the whole wave, in every kind of launch."""
    rng = np.random.default_rng(m)
    lens = rng.integers(0, 12, size=m)
    if kind == "one_long":
        lens[m // 2] = 70001
    elif kind == "many_long":
        lens[rng.random(m) < min(1.0, 3000.0 / m)] = rng.integers(250, 700)
    else:
        lens[:] = 150
        lens[:3] = [0, 257, 1500]
    X, y, w, z = _sparse(lens, 50000)
    _, out = _best_us(X, y, w)
    _check(out, z, w.cpu().numpy().astype(np.float64), 0.01, wl.HINGE)


def test_short_sparse_rows_with_columns_on_both_sides_of_the_head():
    """Times, with a margin of a sixth: four entries to a lane whatever the row's length, each waiting for the one before, took 80 us instead of 59."""
    lens = np.random.default_rng(1).integers(0, 21, 1000000)
    assert _best_us(*_sparse(lens, 30000)[:3])[0] <= 69.0


def test_long_sparse_rows_keep_a_wave_busy():
    """Times, with a margin of a third and of two: 16 lanes to such rows took 71 us instead of 37 (30 for short rows), and
    1530 instead of 322."""
    d = 1 << 20
    few = _best_us(*_sparse(np.full(1000, 3000), d)[:3])[0]
    same_entries = _best_us(*_sparse(np.full(100000, 30), d)[:3])[0]
    assert few <= 1.7 * same_entries, (few, same_entries)
    lens = np.full(200000, 20)
    lens[100000] = 100000
    assert _best_us(*_sparse(lens, d)[:3])[0] <= 650.0


@pytest.mark.parametrize("m,mean,d", [
    (37, 5, 5000), (5000, 3, 5000), (401000, 9, 5000), (401000, 70, 5000),
    (1000, 200, 5000),                            # (a wave to a row)
    (20000, 110, 30000), (401000, 70, 30000),     # columns in the copied head and behind it; rows of 256 entries and of more among them
    (401000, 9, 200000),                          # columns mostly behind the head
    (401000, 29, 5000), (401000, 29, 30000), (401000, 29, 200000)])      # 64 entries and the rest of a row, two to a lane and one
def test_sparse_rows_four_entries_a_lane(m, mean, d):
    """Rows of 0 to 3 * mean entries from any entry of the arrays on, the last one at the arrays' end; the first row_ptr is not zero."""
    rng = np.random.default_rng(m + mean)
    lens = np.minimum(rng.integers(0, 3 * mean, m), rng.integers(0, 3 * mean, m))
    lens[-1] = mean
    if mean == 110:
        lens[5:3000:7] = 256 + np.arange(428) % 3 - 1      # (up to 256 entries 16 lanes, from 257 on the whole wave)
    skip = 3
    row_ptr = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(lens, out=row_ptr[1:])
    nnz = int(row_ptr[-1])
    gap = rng.integers(1, d // (3 * mean), nnz).astype(np.int64)
    total = np.concatenate([[0], np.cumsum(gap)])
    col = (total[1:] - np.repeat(total[row_ptr[:-1]], lens) - 1).astype(np.int32)
    col = np.where(np.repeat(np.arange(m) % 2, lens), d - 1 - col, col).astype(np.int32)      # every other row from the last column down
    val = rng.standard_normal(nnz).astype(np.float32)
    w = rng.standard_normal(d).astype(np.float32)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    cg = torch.from_numpy(np.concatenate([np.full(skip, d - 1, np.int32), col])).cuda()
    vg = torch.from_numpy(np.concatenate([np.full(skip, np.nan, np.float32), val])).cuda()
    X = api.Matrix(m, d, row_ptr=torch.from_numpy(row_ptr + skip).cuda(), col_idx=cg, vals=vg)
    got = api.wpsgd_objective(X, torch.from_numpy(y).cuda(), torch.from_numpy(w).cuda(), 0.1, wl.HINGE).cpu().numpy()
    prod = np.concatenate([[0.0], np.cumsum(w[col].astype(np.float64) * val.astype(np.float64))])
    yhat = prod[row_ptr[1:]] - prod[row_ptr[:-1]]
    ref = 0.05 * float(w.astype(np.float64) @ w) + np.maximum(0.0, 1.0 - y * yhat).mean()
    # running sums of nnz terms of size 1: nnz^1.5 * 1e-16 at most, over the mean of m losses of size 1 and more
    assert abs(got[0] - ref) <= 1e-9 * ref


def test_a_sparse_batch_of_more_than_32_bit_offsets():
    """A row of 2^28 entries: the rows that share its batch go one by one."""
    m, d, n = 4500000, 1000, 1 << 28
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    lens = torch.randint(0, 4, (m,), generator=g, device="cuda", dtype=torch.int64)
    lens[m // 2] = n
    ptr = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=ptr[1:])
    nnz = int(ptr[-1])
    cols = torch.arange(nnz, dtype=torch.int64, device="cuda").remainder_(d).to(torch.int32)
    w = torch.randn(d, generator=g, device="cuda") / 8
    vals = torch.ones(nnz, device="cuda")
    y = torch.where(torch.rand(m, generator=g, device="cuda") < 0.5, 1.0, -1.0)
    out = api.wpsgd_objective(api.Matrix(m, d, row_ptr=ptr, col_idx=cols, vals=vals), y, w, 0.01, wl.HINGE).cpu().numpy()
    w64, p = w.double().cpu().numpy(), ptr.cpu().numpy()
    sums = np.concatenate([[0.0], np.cumsum(w64)])         # w.x of a row: its columns follow each other, round and round
    z = y.double().cpu().numpy() * ((p[1:] // d - p[:-1] // d) * sums[-1] + sums[p[1:] % d] - sums[p[:-1] % d])
    z[p[1:] == p[:-1]] = 0.0
    want = 0.005 * (w64 @ w64) + np.maximum(0.0, 1.0 - z).mean()
    # a lane adds up to 2^22 terms of the long row in fp64, 2^22 * 2^-53 of a sum of 1e6 at most, and the row is one of m
    assert abs(out[0] - want) <= 1e-9 * want
    assert abs(out[1] - (z <= 0).mean()) * m <= 1.0
