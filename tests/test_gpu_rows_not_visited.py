"""Kernels run whole groups of steps; what a group holds behind a chain's last step must not reach the model.  Every row
that no chain visits is NaN here: one of them multiplied by zero and added would show."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

# fp64 state leaves the rounding of the result to fp32 (6e-8 an element); fp32 state a few dozen roundings of it
TOL = {wl.HINGE: 2e-7, wl.LOGISTIC: 5e-6}
PIPE, OCTET = {"block_steps": 16, "prefetch": 7}, {"block_steps": 8}
M, SEED, ETA, LAM = 4000, 9, 0.5, 1e-3


def _visits(n, sampling):
    k = len(n)
    if sampling == api.SAMPLE_SHARDS:
        return [orc.shard_indices(SEED, i, k, 0, int(n[i]), M) for i in range(k)]
    return [orc.sample_indices(SEED, i, 0, int(n[i]), M) for i in range(k)]


def _check(W, X, y, visits, loss):
    for i, idx in enumerate(visits):
        ref, _ = orc.sgd(X, y, idx, ETA, LAM, loss)
        assert np.linalg.norm(W[i] - ref) <= TOL[loss] * max(np.linalg.norm(ref), 1e-30), i


@pytest.mark.parametrize("d,bf16,plan", [
    (50, False, None), (128, True, None), (200, False, {"block_steps": 16}),             # sixteen steps per block
    (1001, False, None), (3001, False, None), (700, True, None), (4096, False, None),    # one workgroup, groups of eight steps
    (16388, False, None), (8200, True, None)])                                           # column slices
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("sampling", [api.SAMPLE_STREAM, api.SAMPLE_SHARDS])
def test_dense_chains(d, bf16, plan, loss, sampling):
    n = np.array([8, 4, 1, 20, 72, 65], dtype=np.int64)
    rng = np.random.default_rng(d)
    visits = _visits(n, sampling)
    seen = np.unique(np.concatenate(visits))
    X = np.full((M, d), math.nan, dtype=np.float32)
    X[seen] = rng.standard_normal((seen.size, d)) / math.sqrt(d)
    y = np.where(rng.random(M) < 0.5, 1.0, -1.0).astype(np.float32)
    dev = torch.from_numpy(X).cuda()
    if bf16:
        dev = dev.to(torch.bfloat16)
        X = dev.float().cpu().numpy()
    W = api.wpsgd_run_chains_from(api.Matrix(M, d, dense=dev), torch.from_numpy(y).cuda(), n, ETA, LAM, loss, SEED, sampling=sampling, plan=plan)
    _check(W.cpu().numpy(), orc.Dense(X), y, visits, loss)


@pytest.mark.parametrize("d,bf16,loss,plan", [
    (50, False, wl.HINGE, PIPE), (64, True, wl.HINGE, PIPE), (50, False, wl.LOGISTIC, PIPE), (128, True, wl.LOGISTIC, PIPE),
    (200, False, wl.LOGISTIC, PIPE), (700, False, wl.LOGISTIC, OCTET), (1024, False, wl.LOGISTIC, OCTET), (2040, True, wl.LOGISTIC, OCTET)])
@pytest.mark.parametrize("sampling", [api.SAMPLE_STREAM, api.SAMPLE_SHARDS])
def test_blocks_that_run_ahead(d, bf16, loss, plan, sampling):
    """Waves and workgroups that prepare blocks reach furthest behind a chain's end."""
    test_dense_chains(d, bf16, plan, loss, sampling)


@pytest.mark.parametrize("per", [7, 40])                       # four steps at a time; one at a time
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("sampling", [api.SAMPLE_STREAM, api.SAMPLE_SHARDS])
def test_sparse_chains(per, loss, sampling):
    d = 30000
    n = np.array([8, 4, 1, 20, 72, 65, 300], dtype=np.int64)
    rng = np.random.default_rng(per)
    visits = _visits(n, sampling)
    seen = np.unique(np.concatenate(visits))
    cols = (np.sort(rng.integers(0, d - per, (M, per)), axis=1) + np.arange(per)).astype(np.int32)         # distinct, ascending
    vals = np.full((M, per), math.nan, dtype=np.float32)
    vals[seen] = rng.standard_normal((seen.size, per)) / math.sqrt(per)
    ptr = np.arange(M + 1, dtype=np.int64) * per
    y = np.where(rng.random(M) < 0.5, 1.0, -1.0).astype(np.float32)
    X = api.Matrix(M, d, row_ptr=torch.from_numpy(ptr).cuda(), col_idx=torch.from_numpy(cols.ravel()).cuda(), vals=torch.from_numpy(vals.ravel()).cuda())
    W = api.wpsgd_run_chains_from(X, torch.from_numpy(y).cuda(), n, ETA, LAM, loss, SEED, sampling=sampling)
    _check(W.cpu().numpy(), orc.CSR(ptr, cols.ravel(), vals.ravel(), d), y, visits, loss)
