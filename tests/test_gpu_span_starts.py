"""Periodic averaging of short rows: the chains of a span form the average of the span before by themselves (those of the block kernels, up
to 63 chains; the first test has both sides of that, the second names the kernel).  Compared, bit for bit, with one call per span and the
averaging entry point between them."""
import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 32, 33, 63, 64])
@pytest.mark.parametrize("d", [4, 5, 63, 64, 66, 128, 252, 256])
@pytest.mark.parametrize("loss,bf16,sampling", [(api.HINGE, False, api.SAMPLE_STREAM), (api.LOGISTIC, False, api.SAMPLE_SHARDS),
                                                (api.LOGISTIC, True, api.SAMPLE_STREAM), (api.HINGE, True, api.SAMPLE_SHARDS)])
def test_spans_of_short_rows_equal_one_call_per_span(k, d, loss, bf16, sampling):
    rng = np.random.default_rng(1000 * k + d)
    m = 70
    X = torch.from_numpy((rng.standard_normal((m, d)) / np.sqrt(d)).astype(np.float32)).cuda()
    X = api.Matrix(m, d, dense=X.to(torch.bfloat16) if bf16 else X)
    y = torch.from_numpy(np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)).cuda()
    steps = rng.integers(0, 40, k).astype(np.int64)         # idle chains among them
    steps[0] = 40
    eta, lam, spans = 0.3, 1e-3, 4
    w = torch.full((d,), 0.01, device="cuda")
    got = api.wpsgd_run_spans(X, y, steps, spans, eta, lam, loss, 11, w_start=w, sampling=sampling)
    a = api.wpsgd_weights(steps, eta, lam)
    for s in range(spans):
        W = api.wpsgd_run_chains_from(X, y, steps, eta, lam, loss, 11, w_start=w, step_offsets=s * steps, sampling=sampling)
        w = api.wpsgd_combine(W, a)
    assert torch.equal(got, w)


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 33, 63, 64])
@pytest.mark.parametrize("d", [4, 63, 65, 66, 68, 127, 128, 129, 130, 132, 252, 255, 256])
@pytest.mark.parametrize("loss", [api.HINGE, api.LOGISTIC])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("plan", [{"block_steps": 16}, {"block_steps": 16, "prefetch": 7}])
def test_starts_of_every_block_kernel(k, d, loss, bf16, plan):
    """One, two and four columns a lane, loads of four columns (whole, and cut by the row's end) and of one; one wave's columns and
    several waves'."""
    if "prefetch" in plan and loss == api.HINGE and d > 64:
        pytest.skip("no such kernel")
    rng = np.random.default_rng(1000 * k + d)
    m = 70
    X = torch.from_numpy((rng.standard_normal((m, d)) / np.sqrt(d)).astype(np.float32)).cuda()
    X = api.Matrix(m, d, dense=X.to(torch.bfloat16) if bf16 else X)
    y = torch.from_numpy(np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)).cuda()
    described = api.wpsgd_describe_plan(X, k, loss, plan)
    assert "scouts=" in described and ("pipelined" in described) == ("prefetch" in plan)
    steps = rng.integers(0, 40, k).astype(np.int64)
    steps[0] = 40
    eta, lam, spans = 0.3, 1e-3, 3
    w = torch.full((d,), 0.01, device="cuda")
    got = api.wpsgd_run_spans(X, y, steps, spans, eta, lam, loss, 11, w_start=w, plan=plan)
    a = api.wpsgd_weights(steps, eta, lam)
    for s in range(spans):
        W = api.wpsgd_run_chains_from(X, y, steps, eta, lam, loss, 11, w_start=w, step_offsets=s * steps, plan=plan)
        w = api.wpsgd_combine(W, a)
    assert torch.equal(got, w)


@pytest.mark.parametrize("k", [1, 15, 16, 17, 63, 64])
@pytest.mark.parametrize("d", [1, 63, 64, 65, 16383, 16384, 16385])
def test_average_of_few_models(k, d):
    """One rounding of an fp64 sum: half a unit in the last place of fp32, and as much again of fp64 per addition."""
    rng = np.random.default_rng(k + d)
    W = rng.standard_normal((k, d)).astype(np.float32)
    a = rng.random(k)
    got = api.wpsgd_combine(torch.from_numpy(W).cuda(), a).cpu().numpy().astype(np.float64)
    want = (a[:, None] * W.astype(np.float64)).sum(axis=0)
    bound = np.abs(want) * 2.0**-24 + (np.abs(a[:, None] * W).sum(axis=0) * k) * 2.0**-52 + 2.0**-149
    assert (np.abs(got - want) <= bound).all()
