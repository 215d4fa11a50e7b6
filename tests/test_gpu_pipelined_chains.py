"""Chains of short rows with everything but the slopes off the dependent path: every way a row, a block, a window or a
chain can end, against the oracle.  (The plan names the kernel: left to choose, calls of few steps run others.)"""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

STEPS = np.array([0, 1, 15, 16, 17, 47, 48, 63, 64, 65, 128, 333], dtype=np.int64)
# fp64 state leaves the rounding of the result to fp32 (6e-8 an element); fp32 state some 300 roundings of it
TOL = {wl.HINGE: 2e-7, wl.LOGISTIC: 2e-5}
PIPE = {"block_steps": 16, "prefetch": 7}
SHAPES = [(wl.HINGE, b, d) for b in (False, True) for d in (4, 5, 16, 31, 63, 64)] + \
         [(wl.LOGISTIC, b, d) for b in (False, True) for d in (4, 7, 17, 64, 65, 98, 128, 129, 191, 255, 256)]


def _data(m, d, bf16, seed):
    rng = np.random.default_rng(seed)
    X = (rng.standard_normal((m, d)) / math.sqrt(d)).astype(np.float32)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    if bf16:
        bits = wl.f32_to_bf16_bits(X)
        return bits, torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16), y
    return X, torch.from_numpy(X).cuda(), y


def _compare(W, ref, tol):
    for i in range(len(ref)):
        assert np.linalg.norm(W[i] - ref[i]) <= tol * max(np.linalg.norm(ref[i]), 1e-30), i


@pytest.mark.parametrize("loss,bf16,d", SHAPES)
def test_every_row_end_and_chain_end(loss, bf16, d):
    host, dev, y = _data(200, d, bf16, d + 7 * loss)
    X, yg = api.Matrix(200, d, dense=dev), torch.from_numpy(y).cuda()
    assert "long=pipelined" in api.wpsgd_describe_plan(X, len(STEPS), loss)
    W = api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, loss, 9, plan=PIPE)
    _compare(W.cpu().numpy(), orc.run_chains(orc.Dense(host), y, STEPS, 0.5, 1e-3, loss, 9)[0], TOL[loss])
    assert torch.equal(W, api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, loss, 9, plan=PIPE))


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("sampling", [api.SAMPLE_STREAM, api.SAMPLE_SHARDS])
def test_start_vector_offsets_and_shards(loss, sampling):
    d, m = 61, 61                                 # shares of five or six rows: a block runs round them several times
    host, dev, y = _data(m, d, False, 5)
    X, yg = api.Matrix(m, d, dense=dev), torch.from_numpy(y).cuda()
    w0 = torch.linspace(-1.0, 1.0, d, device="cuda")
    off = np.arange(len(STEPS), dtype=np.int64) * 37
    args = (X, yg, STEPS, 0.3, 1e-2, loss, 3)
    W = api.wpsgd_run_chains_from(*args, w_start=w0, step_offsets=off, sampling=sampling, plan=PIPE)
    other = api.wpsgd_run_chains_from(*args, w_start=w0, step_offsets=off, sampling=sampling,
                                      plan={"threads": 64, "block_steps": 1, "prefetch": 8})
    _compare(W.cpu().numpy(), other.cpu().numpy().astype(np.float64), TOL[loss])
    assert torch.equal(W[0], w0)


@pytest.mark.parametrize("d", [40, 130])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_scale_is_folded_at_every_window(d, loss):
    """eta*lambda = 0.4: the scale falls below 2^-30 within a window, so that a block's products with the block before
    cross a folding.  250 chains: one to a compute unit."""
    k = 250
    host, dev, y = _data(64, d, False, 8)
    n = np.resize(STEPS, k)
    X, yg = api.Matrix(64, d, dense=dev), torch.from_numpy(y).cuda()
    W = api.wpsgd_run_chains(X, yg, n, 0.8, 0.5, loss, 4, plan=PIPE if loss == wl.LOGISTIC or d <= 64 else None).cpu().numpy()
    _compare(W[:24], orc.run_chains(orc.Dense(host), y, n, 0.8, 0.5, loss, 4, chain_ids=np.arange(24))[0], TOL[loss])
    _compare(W[-12:], orc.run_chains(orc.Dense(host), y, n, 0.8, 0.5, loss, 4, chain_ids=np.arange(k - 12, k))[0], TOL[loss])


@pytest.mark.parametrize("loss,d", [(wl.HINGE, 33), (wl.HINGE, 64), (wl.LOGISTIC, 33), (wl.LOGISTIC, 128), (wl.LOGISTIC, 200)])
def test_rows_that_are_not_finite(d, loss):
    """From the step that meets an infinity on, the model holds infinities or NaN; which ones, and where the rest of it
    stands still, is as with one step at a time."""
    m, k = 300, 40
    rng = np.random.default_rng(d)
    host = (rng.standard_normal((m, d)) / math.sqrt(d)).astype(np.float32)
    bad = rng.choice(m, 12, replace=False)
    host[bad, rng.integers(0, d, 12)] = np.resize(np.array([math.inf, -math.inf, math.nan], dtype=np.float32), 12)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    w0 = rng.standard_normal(d).astype(np.float32)
    n = np.full(k, 45, dtype=np.int64)
    n[-1] = 200
    W = api.wpsgd_run_chains_from(api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, 0.5, 1e-3, loss, 9,
                                  w_start=torch.from_numpy(w0).cuda(), plan=PIPE).cpu().numpy()
    spoiled = 0
    with np.errstate(invalid="ignore"):
        for i in range(k):
            ref, _ = orc.sgd(orc.Dense(host), y, orc.sample_indices(9, i, 0, int(n[i]), m), 0.5, 1e-3, loss, w0=w0.astype(np.float64))
            spoiled += not np.isfinite(ref).all()
            # elementwise: a few dozen fp32 roundings of the model's entries, whose size is 1 (logistic); one (hinge)
            np.testing.assert_allclose(W[i], ref, rtol=1e-5, atol=1e-5 if loss == wl.LOGISTIC else 2e-7, equal_nan=True)
    assert 10 <= spoiled <= k


@pytest.mark.parametrize("d", [64, 128])
def test_rows_of_very_different_size(d):
    """Rows of 1e17 an element among rows of 0.1: products of 1e36, 1e18 and 1 in one block."""
    m, k = 100, 9
    host, _, y = _data(m, d, False, d)
    host[::7] *= np.float32(1e18)
    n = np.full(k, 200, dtype=np.int64)
    args = (api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, 0.5, 1e-3, wl.LOGISTIC, 9)
    W = api.wpsgd_run_chains(*args).cpu().numpy()
    other = api.wpsgd_run_chains(*args, plan={"threads": 64, "block_steps": 1, "prefetch": 8}).cpu().numpy()
    assert np.isfinite(other).all() and np.abs(other).max() > 1e15
    for i in range(k):            # after a step of 1e17 an element nothing else is left of the model: a few roundings of the largest
        assert np.abs(W[i] - other[i]).max() <= 1e-4 * np.abs(other[i]).max(), i


@pytest.mark.parametrize("d", [64, 128, 200])
@pytest.mark.parametrize("size,eta", [(1e20, 0.5), (1e19, 8.0)])
def test_rows_too_large_for_products(d, size, eta):
    """Finite rows whose fp32 products overflow (1e20), or whose products do with a step's coefficient on them (1e19).  Large rows share a
    direction and have no element below zero, so that v.x may be infinite but is never a NaN one step at a time."""
    m, k = 100, 9
    rng = np.random.default_rng(d)
    host, _, y = _data(m, d, False, d)
    u = np.abs(rng.standard_normal(d))
    host[::4] = (size * u / np.linalg.norm(u)).astype(np.float32)
    n = np.full(k, 200, dtype=np.int64)
    pairs = 0                     # of large rows in a block
    for i in range(k):
        blocks = (orc.sample_indices(9, i, 0, 200, m) % 4 == 0)[:200 // 16 * 16].reshape(-1, 16).sum(axis=1)
        pairs += int((blocks * (blocks - 1) // 2).sum())
    product, most = float(host[0].astype(np.float64) @ host[0]), float(np.finfo(np.float32).max)
    assert pairs >= 100 and (product > 2 * most if size == 1e20 else 0.25 * most < product < 0.5 * most and eta * product / math.log(2) > 2 * most)
    args = (api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, eta, 1e-3, wl.LOGISTIC, 9)
    W = api.wpsgd_run_chains(*args, plan=PIPE).cpu().numpy()
    other = api.wpsgd_run_chains(*args, plan={"threads": 64, "block_steps": 1, "prefetch": 8}).cpu().numpy()
    assert np.isfinite(other).all() and np.abs(other).max() > 1e17
    for i in range(k):            # after a step of that size nothing else is left of the model: a few roundings of the largest
        assert np.abs(W[i] - other[i]).max() <= 1e-4 * np.abs(other[i]).max(), i
