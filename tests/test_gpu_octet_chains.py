"""Logistic chains of longer rows, eight steps per block, whose products between rows other workgroups form: every way a row, a block, a
window or a chain can end, against the oracle.  (The longest chain of a call decides whether this kernel runs: see the planner.)"""
import math
import time

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

STEPS = np.array([0, 1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 72, 128, 333], dtype=np.int64)
TOL = 2e-5                         # fp32 state: some 300 roundings of 6e-8 an element
SHAPES = [(False, d) for d in (513, 514, 515, 767, 1001, 1022, 1023, 1024)] + \
         [(True, d) for d in (520, 1016, 1024, 2040, 2048)]


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


@pytest.mark.parametrize("bf16,d", SHAPES)
def test_every_row_end_and_chain_end(bf16, d):
    host, dev, y = _data(200, d, bf16, d)
    X, yg = api.Matrix(200, d, dense=dev), torch.from_numpy(y).cuda()
    assert "long=octets" in api.wpsgd_describe_plan(X, len(STEPS), wl.LOGISTIC)
    W = api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, wl.LOGISTIC, 9)
    _compare(W.cpu().numpy(), orc.run_chains(orc.Dense(host), y, STEPS, 0.5, 1e-3, wl.LOGISTIC, 9)[0], TOL)


@pytest.mark.parametrize("d", [513, 700, 1024])
def test_results_do_not_depend_on_the_helpers(d):
    """Three helpers a chain, two, one and none: a chain of the same number takes the same steps and has the same bits, whichever
    products were there in time."""
    _, dev, y = _data(500, d, False, d)
    X, yg = api.Matrix(500, d, dense=dev), torch.from_numpy(y).cuda()
    runs = []
    for k, plan in ((6, None), (6, None), (48, None), (64, None), (6, {"block_steps": 8, "helpers": 1}), (6, {"block_steps": 8, "helpers": -1})):
        n = np.full(k, 700, dtype=np.int64)
        runs.append(api.wpsgd_run_chains(X, yg, n, 0.5, 1e-3, wl.LOGISTIC, 9, plan=plan)[:6])
    for W in runs[1:]:
        assert torch.equal(W, runs[0])


@pytest.mark.parametrize("sampling", [api.SAMPLE_STREAM, api.SAMPLE_SHARDS])
def test_start_vector_offsets_shards_and_row_stride(sampling):
    d, m = 601, 61                                # shares of four or five rows: a block runs round them
    host, _, y = _data(m, d, False, 5)
    padded = torch.zeros((m, d + 6), device="cuda")
    padded[:, :d] = torch.from_numpy(host).cuda()
    X, yg = api.Matrix(m, d, dense=padded[:, :d]), torch.from_numpy(y).cuda()
    w0 = torch.linspace(-1.0, 1.0, d, device="cuda")
    off = np.arange(len(STEPS), dtype=np.int64) * 37
    args = (X, yg, STEPS, 0.3, 1e-2, wl.LOGISTIC, 3)
    W = api.wpsgd_run_chains_from(*args, w_start=w0, step_offsets=off, sampling=sampling)
    other = api.wpsgd_run_chains_from(*args, w_start=w0, step_offsets=off, sampling=sampling,
                                      plan={"threads": 256, "block_steps": 1})
    _compare(W.cpu().numpy(), other.cpu().numpy().astype(np.float64), TOL)
    assert torch.equal(W[0], w0)


def test_spans_are_runs_one_after_the_other():
    d, m, k = 520, 300, 10
    _, dev, y = _data(m, d, False, 6)
    X, yg = api.Matrix(m, d, dense=dev), torch.from_numpy(y).cuda()
    n = np.arange(k, dtype=np.int64) * 9 + 120
    w = None
    for s in range(4):
        W = api.wpsgd_run_chains_from(X, yg, n, 0.4, 1e-3, wl.LOGISTIC, 3, w_start=w, step_offsets=n * s)
        w = api.wpsgd_combine(W, api.wpsgd_weights(n, 0.4, 1e-3))
    assert torch.equal(api.wpsgd_run_spans(X, yg, n, 4, 0.4, 1e-3, wl.LOGISTIC, 3), w)


@pytest.mark.parametrize("d", [600, 1001])
def test_scale_is_folded_at_every_window(d):
    """eta*lambda = 0.4: the scale falls below 2^-30 within a window."""
    host, dev, y = _data(64, d, False, 8)
    X, yg = api.Matrix(64, d, dense=dev), torch.from_numpy(y).cuda()
    W = api.wpsgd_run_chains(X, yg, STEPS, 0.8, 0.5, wl.LOGISTIC, 4).cpu().numpy()
    _compare(W, orc.run_chains(orc.Dense(host), y, STEPS, 0.8, 0.5, wl.LOGISTIC, 4)[0], TOL)


@pytest.mark.parametrize("d", [513, 1024])
def test_rows_that_are_not_finite(d):
    """From the step that meets an infinity on, the model holds infinities or NaN; which ones, and where the rest of it
    stands still, is as with one step at a time."""
    m, k = 300, 30                                # (up to 32 chains, blocks of eight from 192 steps on)
    rng = np.random.default_rng(d)
    host = (rng.standard_normal((m, d)) / math.sqrt(d)).astype(np.float32)
    bad = rng.choice(m, 12, replace=False)
    host[bad, rng.integers(0, d, 12)] = np.resize(np.array([math.inf, -math.inf, math.nan], dtype=np.float32), 12)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    w0 = rng.standard_normal(d).astype(np.float32)
    n = np.full(k, 45, dtype=np.int64)
    n[-1] = 200
    W = api.wpsgd_run_chains_from(api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, 0.5, 1e-3, wl.LOGISTIC, 9,
                                  w_start=torch.from_numpy(w0).cuda()).cpu().numpy()
    spoiled = 0
    with np.errstate(invalid="ignore"):
        for i in range(k):
            ref, _ = orc.sgd(orc.Dense(host), y, orc.sample_indices(9, i, 0, int(n[i]), m), 0.5, 1e-3, wl.LOGISTIC, w0=w0.astype(np.float64))
            spoiled += not np.isfinite(ref).all()
            # elementwise: a few dozen fp32 roundings of the model's entries, whose size is 1
            np.testing.assert_allclose(W[i], ref, rtol=1e-5, atol=1e-5, equal_nan=True)
    assert 10 <= spoiled <= k


def test_rows_of_very_different_size():
    """Rows of 1e17 an element among rows of 0.1: products of 1e36, 1e18 and 1 in one block."""
    m, k, d = 100, 9, 520
    host, _, y = _data(m, d, False, d)
    host[::7] *= np.float32(1e18)
    n = np.full(k, 200, dtype=np.int64)
    args = (api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, 0.5, 1e-3, wl.LOGISTIC, 9)
    W = api.wpsgd_run_chains(*args).cpu().numpy()
    other = api.wpsgd_run_chains(*args, plan={"threads": 256, "block_steps": 1}).cpu().numpy()
    assert np.isfinite(other).all() and np.abs(other).max() > 1e15
    for i in range(k):            # after a step of 1e17 an element nothing else is left of the model: a few roundings of the largest
        assert np.abs(W[i] - other[i]).max() <= 1e-4 * np.abs(other[i]).max(), i


def _us_of_calls(X, yg, k, n, plan, streams):
    steps = np.full(k, n, dtype=np.int64)
    ws = [torch.empty(api.wpsgd_run_chains_workspace(X, k, wl.LOGISTIC, plan), dtype=torch.uint8, device="cuda") for _ in streams]
    W = [torch.empty((k, X.d), device="cuda") for _ in streams]
    times = []
    for _ in range(11):
        torch.cuda.synchronize()
        start = time.perf_counter()
        for i, s in enumerate(streams):
            api.wpsgd_run_chains(X, yg, steps, 0.05, 1e-4, wl.LOGISTIC, 9 + i, W=W[i], workspace=ws[i], plan=plan, stream=s)
        torch.cuda.synchronize()
        times.append((time.perf_counter() - start) * 1e6)
    return sorted(times)[5]


@pytest.mark.parametrize("k", [16, 64, 80])
def test_helpers_leave_room_for_a_call_on_another_stream(k):
    """Times: with helpers on every compute unit two calls of 64 chains took 14 % longer than two calls without (and 12 % less as it is)."""
    _, dev, y = _data(8000, 1024, False, 1)
    X, yg = api.Matrix(8000, 1024, dense=dev), torch.from_numpy(y).cuda()
    none = {"helpers": -1}
    for _ in range(4):                            # (some pairs of streams share a hardware queue, and nothing overlaps)
        streams = [torch.cuda.Stream() for _ in range(2)]
        alone = _us_of_calls(X, yg, k, 4000, none, streams)
        if alone < 1.6 * _us_of_calls(X, yg, k, 4000, none, streams[:1]):
            break
    helped = _us_of_calls(X, yg, k, 4000, None, streams)
    assert helped <= 1.08 * alone, (helped, alone)


def _us_per_step(X, yg, k, n):
    steps = np.full(k, n, dtype=np.int64)
    best = float("inf")
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        api.wpsgd_run_chains(X, yg, steps, 0.05, 1e-4, wl.LOGISTIC, 9)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


@pytest.mark.parametrize("bf16,d", [(False, 1024), (True, 2048)])
def test_helpers_stay_with_a_long_chain(bf16, d):
    """Times: helpers that left a chain of 1.5 million steps on the way made its steps 15 % (fp32) and 30 % (bf16) slower on average."""
    _, dev, y = _data(2000, d, bf16, 1)
    X, yg = api.Matrix(2000, d, dense=dev), torch.from_numpy(y).cuda()
    usual, long = _us_per_step(X, yg, 8, 200000), _us_per_step(X, yg, 8, 1500000)
    assert long <= 1.07 * usual, (long, usual)


@pytest.mark.parametrize("size,eta", [(1e20, 0.5), (1e19, 8.0)])
def test_rows_too_large_for_products(size, eta):
    """Finite rows whose fp32 products overflow (1e20), or whose products do with a step's coefficient on them (1e19).  Large rows share a
    direction and have no element below zero, so that v.x may be infinite but is never a NaN one step at a time."""
    m, k, d = 100, 9, 520
    rng = np.random.default_rng(d)
    host, _, y = _data(m, d, False, d)
    u = np.abs(rng.standard_normal(d))
    host[::4] = (size * u / np.linalg.norm(u)).astype(np.float32)
    n = np.full(k, 200, dtype=np.int64)
    pairs = 0                     # of large rows in a block
    for i in range(k):
        blocks = (orc.sample_indices(9, i, 0, 200, m) % 4 == 0)[:200 // 8 * 8].reshape(-1, 8).sum(axis=1)
        pairs += int((blocks * (blocks - 1) // 2).sum())
    product, most = float(host[0].astype(np.float64) @ host[0]), float(np.finfo(np.float32).max)
    assert pairs >= 100 and (product > 2 * most if size == 1e20 else 0.25 * most < product < 0.5 * most and eta * product / math.log(2) > 2 * most)
    args = (api.Matrix(m, d, dense=torch.from_numpy(host).cuda()), torch.from_numpy(y).cuda(), n, eta, 1e-3, wl.LOGISTIC, 9)
    W = api.wpsgd_run_chains(*args, plan={"block_steps": 8}).cpu().numpy()
    other = api.wpsgd_run_chains(*args, plan={"threads": 256, "block_steps": 1}).cpu().numpy()
    assert np.isfinite(other).all() and np.abs(other).max() > 1e17
    for i in range(k):            # after a step of that size nothing else is left of the model: a few roundings of the largest
        assert np.abs(W[i] - other[i]).max() <= 1e-4 * np.abs(other[i]).max(), i


def test_workspace_without_room_for_records():
    """The register kernels need no room behind the header and the shuffled order: a call that brings only that is still served."""
    d, m = 1024, 100
    host, dev, y = _data(m, d, False, 2)
    X, yg = api.Matrix(m, d, dense=dev), torch.from_numpy(y).cuda()
    whole = api.wpsgd_run_chains_workspace(X, len(STEPS), wl.LOGISTIC)
    ws = torch.empty(whole - len(STEPS) * d * 4, dtype=torch.uint8, device="cuda")
    with pytest.raises(api.WpsgdError) as err:             # (but a plan that names the kernel is not given another)
        api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, wl.LOGISTIC, 9, workspace=ws, plan={"block_steps": 8})
    assert err.value.status == api.WORKSPACE_TOO_SMALL
    W = api.wpsgd_run_chains(X, yg, STEPS, 0.5, 1e-3, wl.LOGISTIC, 9, workspace=ws)
    _compare(W.cpu().numpy(), orc.run_chains(orc.Dense(host), y, STEPS, 0.5, 1e-3, wl.LOGISTIC, 9)[0], TOL)
