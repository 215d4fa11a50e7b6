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
