"""The weighted average is a chain of fused multiply-adds in fp64, in the order of the models: no product is rounded by itself.
The models cancel, so that one rounding more or less is the whole result; compared bit for bit with a chain formed by exact fractions."""
from fractions import Fraction

import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api

pytestmark = pytest.mark.gpu


def _fused(W, a):
    """fp32 of acc = fma(a[i], W[i], acc), one column"""
    acc = 0.0
    for x, w in zip(W, a):
        acc = float(Fraction(float(w)) * Fraction(float(x)) + Fraction(acc))      # (a float from a fraction is rounded once)
    return np.float32(acc)


@pytest.mark.parametrize("k", [2, 15, 16, 17, 33, 63])
@pytest.mark.parametrize("d", [5, 64, 16384, 16385, 16388])
def test_products_are_not_rounded(k, d):
    rng = np.random.default_rng(k + d)
    base = rng.standard_normal(40).astype(np.float32)
    W = np.zeros((k, 40), dtype=np.float32)
    a = np.zeros(k)
    for i in range(0, k - 1, 2):                  # pairs of equal weights and opposite models
        W[i], W[i + 1] = base * np.float32(i + 1), -base * np.float32(i + 1)
        a[i] = a[i + 1] = rng.random()
    want = np.array([_fused(W[:, c], a) for c in range(40)])
    assert (want != 0.0).sum() > 10               # (rounded products cancel to zero)
    got = api.wpsgd_combine(torch.from_numpy(np.tile(W, (1, d // 40 + 1))[:, :d].copy()).cuda(), a).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), np.tile(want, d // 40 + 1)[:d].view(np.uint32))


@pytest.mark.parametrize("plan", [{"block_steps": 16}, {"block_steps": 16, "prefetch": 7}])
@pytest.mark.parametrize("d", [8, 63, 66, 128, 129, 252, 256])
@pytest.mark.parametrize("loss,bf16", [(api.HINGE, False), (api.HINGE, True), (api.LOGISTIC, False), (api.LOGISTIC, True)])
def test_chains_that_average_for_themselves(plan, d, loss, bf16):
    """Three chains with one row each, x, -x and 0: the models cancel up to the roundings of the average, and the next span starts there."""
    if "prefetch" in plan and loss == api.HINGE and d > 64:
        pytest.skip("no such kernel")
    rng = np.random.default_rng(d)
    x = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    X = torch.from_numpy(np.stack([x, np.zeros_like(x), -x])).cuda()
    X = api.Matrix(3, d, dense=X.to(torch.bfloat16) if bf16 else X)
    y = torch.ones(3, device="cuda")
    steps = np.full(3, 20, dtype=np.int64)
    eta, lam, spans = 0.3, 1e-3, 3
    described = api.wpsgd_describe_plan(X, 3, loss, plan)
    assert "scouts=" in described and ("pipelined" in described) == ("prefetch" in plan)
    got = api.wpsgd_run_spans(X, y, steps, spans, eta, lam, loss, 11, sampling=api.SAMPLE_SHARDS, plan=plan)
    a = api.wpsgd_weights(steps, eta, lam)
    w = torch.zeros(d, device="cuda")
    for s in range(spans):
        W = api.wpsgd_run_chains_from(X, y, steps, eta, lam, loss, 11, w_start=w, step_offsets=s * steps, sampling=api.SAMPLE_SHARDS, plan=plan)
        w = api.wpsgd_combine(W, a)
    assert torch.equal(got, w)
    assert 0.0 < float(w.abs().max()) < 1e-6
