"""Chains of short rows, sixteen steps per block: every way a row, a block or a window can end, against the oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

BLOCK = {"block_steps": 16}
STEPS = np.array([0, 1, 15, 16, 17, 47, 48, 63, 64, 65, 128, 300], dtype=np.int64)


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


# fp64 state leaves the rounding of the result to fp32 (6e-8 an element); fp32 state some 300 roundings of it
TOL = {wl.HINGE: 2e-7, wl.LOGISTIC: 2e-5}


@pytest.mark.parametrize("d", [4, 5, 15, 16, 17, 31, 63, 64, 65, 98, 127, 128, 129, 191, 255, 256])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_every_row_end_and_chain_end(d, bf16, loss):
    host, dev, y = _data(200, d, bf16, d + 7 * loss)
    X = api.Matrix(200, d, dense=dev)
    yg = torch.from_numpy(y).cuda()
    assert ("scouts=3" in api.wpsgd_describe_plan(X, len(STEPS), loss)) == (d <= 128 or bf16 or loss == wl.LOGISTIC)
    forced = api.wpsgd_describe_plan(X, len(STEPS), loss, BLOCK)
    assert "B=16 P=2" in forced and "pipelined" not in forced                   # (the pipeline has tests of its own)
    W = api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, loss, 9, plan=BLOCK)
    ref = orc.run_chains(orc.Dense(host), y, STEPS, 0.5, 1e-3, loss, 9)[0]
    _compare(W.cpu().numpy(), ref, TOL[loss])
    assert torch.equal(W, api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, loss, 9, plan=BLOCK))


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
@pytest.mark.parametrize("sampling", [api.SAMPLE_STREAM, api.SAMPLE_SHARDS])
def test_start_vector_offsets_and_shards(loss, sampling):
    d, m = 77, 61                                 # shares of five or six rows: a block runs round them several times
    host, dev, y = _data(m, d, False, 5)
    X, yg = api.Matrix(m, d, dense=dev), torch.from_numpy(y).cuda()
    w0 = torch.linspace(-1.0, 1.0, d, device="cuda")
    off = np.arange(len(STEPS), dtype=np.int64) * 37
    W = api.wpsgd_run_chains_from(X, yg, STEPS, 0.3, 1e-2, loss, 3, w_start=w0, step_offsets=off, sampling=sampling, plan=BLOCK)
    other = api.wpsgd_run_chains_from(X, yg, STEPS, 0.3, 1e-2, loss, 3, w_start=w0, step_offsets=off, sampling=sampling,
                                      plan={"threads": 64, "block_steps": 1, "prefetch": 8})
    _compare(W.cpu().numpy(), other.cpu().numpy().astype(np.float64), TOL[loss])
    assert torch.equal(W[0], w0)


@pytest.mark.parametrize("d", [33, 128, 200])
@pytest.mark.parametrize("shift", [20, 40, 54])
def test_large_rows_stay_in_blocks(d, shift):
    """Rows 2^s times as large, eta 2^-2s and lambda 2^2s times: the models are 2^-s times as large, bit for bit, unless the blocks
    give up on rows that large and take one step after the other, whose sums have another order."""
    _, dev, y = _data(200, d, False, d)
    yg, s = torch.from_numpy(y).cuda(), 2.0 ** shift
    W = api.wpsgd_run_chains(api.Matrix(200, d, dense=dev), yg, STEPS, 0.5, 1e-3, wl.LOGISTIC, 9, plan=BLOCK)
    scaled = api.wpsgd_run_chains(api.Matrix(200, d, dense=dev * s), yg, STEPS, 0.5 / (s * s), 1e-3 * (s * s), wl.LOGISTIC, 9, plan=BLOCK)
    assert torch.equal(scaled * s, W)


@pytest.mark.parametrize("d,e", [(33, 54), (200, 52)])
def test_large_rows_and_a_large_eta(d, e):
    """Products between rows that are finite and, with a step's coefficient, are not: the first step moves the model by half of eta, to
    where no later one moves it, and a slope of 0 times such a product must stay 0."""
    rng = np.random.default_rng(d)
    y = np.where(rng.random(100) < 0.5, 1.0, -1.0).astype(np.float32)
    host = np.repeat(y[:, None] * np.float32(2.0 ** e), d, axis=1)
    product = np.float32(d * 4.0 ** e)
    eta = 2.0 ** 127.57 / float(product)
    with np.errstate(over="ignore"):
        assert np.isfinite(product * np.float32(0.5 * eta / math.log(2))) and np.isinf(product * np.float32(eta / math.log(2)))
    n = np.full(9, 48, dtype=np.int64)
    args = (api.Matrix(100, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, eta, 0.0, wl.LOGISTIC, 9)
    W = api.wpsgd_run_chains(*args, plan=BLOCK).cpu().numpy()
    np.testing.assert_allclose(W, np.full((9, d), 0.5 * eta * 2.0 ** e), rtol=1e-6)            # (a handful of fp32 roundings)


@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_scale_is_folded_and_many_chains_run(loss):
    """eta*lambda = 0.4: the scale falls below 2^-30 within a window.  900 chains: several to a compute unit."""
    d, k = 130, 900
    host, dev, y = _data(64, d, False, 8)
    n = np.resize(STEPS, k)
    X, yg = api.Matrix(64, d, dense=dev), torch.from_numpy(y).cuda()
    W = api.wpsgd_run_chains(X, yg, n, 0.8, 0.5, loss, 4, plan=BLOCK).cpu().numpy()
    ref = orc.run_chains(orc.Dense(host), y, n, 0.8, 0.5, loss, 4, chain_ids=np.arange(24))[0]
    _compare(W[:24], ref, TOL[loss])
    _compare(W[-12:], orc.run_chains(orc.Dense(host), y, n, 0.8, 0.5, loss, 4, chain_ids=np.arange(k - 12, k))[0], TOL[loss])


@pytest.mark.parametrize("d", [33, 128, 200])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
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
    W = api.wpsgd_run_chains_from(api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, 0.5, 1e-3, loss, 9,
                                  w_start=torch.from_numpy(w0).cuda(), plan=BLOCK).cpu().numpy()
    spoiled = 0
    with np.errstate(invalid="ignore"):
        for i in range(k):
            ref, _ = orc.sgd(orc.Dense(host), y, orc.sample_indices(9, i, 0, 45, m), 0.5, 1e-3, loss, w0=w0.astype(np.float64))
            spoiled += not np.isfinite(ref).all()
            # elementwise: a few dozen fp32 roundings of the model's entries, whose size is 1 (logistic); one (hinge)
            np.testing.assert_allclose(W[i], ref, rtol=1e-5, atol=1e-5 if loss == wl.LOGISTIC else 2e-7, equal_nan=True)
    assert 10 <= spoiled < k
