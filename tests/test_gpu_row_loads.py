"""Rows that are not 16-byte aligned: fp32 rows are fetched four dwords at a time whatever their length,
stride and base, so what lies behind a row's last column must never reach the result."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

K_STEPS = np.array([130, 0, 1, 65, 64], dtype=np.int64)
# fp64 state leaves the rounding of the result to fp32 (6e-8 an element); fp32 state some 130 roundings of the model and of its products
TOL = {wl.HINGE: 2e-7, wl.LOGISTIC: 1e-5}


def _embedded(X, ld, shift):
    """X as a view with row stride ld whose base lies `shift` elements behind a 256-byte boundary; NaN all around."""
    m, d = X.shape
    flat = torch.full((m * ld + shift + 8,), math.nan, dtype=torch.float32, device="cuda")
    view = flat[shift:shift + m * ld].view(m, ld)[:, :d]
    view.copy_(torch.from_numpy(X))
    return flat, api.Matrix(m, d, dense=view)


@pytest.mark.parametrize("d,ld,shift", [
    (1, 1, 0), (3, 5, 1), (63, 63, 2), (65, 66, 3), (101, 101, 0), (254, 255, 1), (257, 257, 1), (515, 515, 2),
    (1023, 1025, 3), (1297, 1297, 0), (2049, 2050, 1), (3001, 3001, 0), (4093, 4093, 1), (4095, 4096, 0), (8190, 8191, 2),
    (16387, 16387, 1)])                                    # the last one: column slices
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_rows_at_any_dword(d, ld, shift, loss):
    rng = np.random.default_rng(d * 3 + loss)
    m = 128
    X = (rng.standard_normal((m, d)) / math.sqrt(d)).astype(np.float32)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    flat, Xg = _embedded(X, ld, shift)
    yg = torch.from_numpy(y).cuda()
    W = api.wpsgd_run_chains(Xg, yg, K_STEPS, 0.5, 1e-3, loss, 9)
    ref = orc.run_chains(orc.Dense(X), y, K_STEPS, 0.5, 1e-3, loss, 9)
    ref = ref[0] if isinstance(ref, tuple) else ref
    got = W.cpu().numpy()
    for i in range(len(K_STEPS)):
        scale = max(np.linalg.norm(ref[i]), 1e-30)
        assert np.linalg.norm(got[i] - ref[i]) <= TOL[loss] * scale, (d, ld, shift, i)
    # the objective reads rows and model with the same kind of load; its sums are fp64 (order of the sum only)
    out = api.wpsgd_objective(Xg, yg, W[0].contiguous(), 1e-3, loss).cpu().numpy()
    w = got[0].astype(np.float64)
    z = y * (X.astype(np.float64) @ w)
    l = np.maximum(0.0, 1.0 - z) if loss == wl.HINGE else np.logaddexp(0.0, -z)
    assert abs(out[0] - (0.5e-3 * (w @ w) + l.mean())) <= 1e-11 * max(1.0, abs(out[0]))
    assert abs(out[1] - (z <= 0).mean()) <= 1.0 / m


@pytest.mark.parametrize("d", [480, 501, 512, 520, 1000, 1001, 1024, 1032, 2001, 2048, 4001, 4096])
@pytest.mark.parametrize("k", [5, 300])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_bf16_rows_on_every_workgroup_size(d, k, loss):
    """Few chains and many take different workgroup sizes and steps per round; both match the oracle."""
    rng = np.random.default_rng(d * 5 + loss)
    m = 96
    bits = wl.f32_to_bf16_bits((rng.standard_normal((m, d)) / math.sqrt(d)).astype(np.float32))
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    n = np.resize(K_STEPS, k)
    Xg = api.Matrix(m, d, dense=torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16))
    W = api.wpsgd_run_chains(Xg, torch.from_numpy(y).cuda(), n, 0.5, 1e-3, loss, 9).cpu().numpy()
    ids = np.array([0, 1, 2, 3, 4, k - 1])
    ref = orc.run_chains(orc.Dense(bits), y, n, 0.5, 1e-3, loss, 9, chain_ids=ids)[0]
    for q, i in enumerate(ids):
        assert np.linalg.norm(W[i] - ref[q]) <= TOL[loss] * max(np.linalg.norm(ref[q]), 1e-30), (d, k, i)


@pytest.mark.parametrize("d", [50, 333, 542, 1023, 2047, 4095])
@pytest.mark.parametrize("tau", [0, 1, 4])
@pytest.mark.parametrize("check", [True, False])
def test_delay_servers_on_rows_at_any_dword(d, tau, check):
    """fp32 rows without 16-byte alignment take the register kernel of the servers; NaN around the rows shows a
    column too many.  fp64 state: only the rounding of W is left (6e-8 an element)."""
    w = wl.delay_servers(m=150, d=d, k=5, n_lo=1, n_hi=60)
    flat, Xg = _embedded(w.dense, d + 2, 1)
    Wg, acc = api.wpsgd_run_delay_chains(Xg, torch.from_numpy(w.y).cuda(), w.n_steps, w.eta, w.lam, w.loss, w.seed, tau, check=check,
                                         w_start=torch.from_numpy(w.meta["w_start"]).cuda())
    for i in range(w.k):
        idx = orc.sample_indices(w.seed, i, 0, int(w.n_steps[i]), w.m)
        ref, acc_o, gap = orc.delay_sgd(orc.Dense(w.dense), w.y, idx, w.eta, w.lam, w.loss, tau,
                                        w0=w.meta["w_start"].astype(np.float64), check=check)
        if gap < 1e-12:
            continue
        assert int(acc[i]) == acc_o, (d, tau, check, i)
        assert np.linalg.norm(Wg[i].cpu().numpy() - ref) <= 2e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("d,bf16", [(8200, True), (12000, True), (16384, True), (16388, False), (24001, False), (33000, False), (65536, False)])
@pytest.mark.parametrize("loss", [wl.HINGE, wl.LOGISTIC])
def test_column_slices_of_either_workgroup_size(d, bf16, loss):
    rng = np.random.default_rng(d + loss)
    m = 70
    X = (rng.standard_normal((m, d)) / math.sqrt(d)).astype(np.float32)
    y = np.where(rng.random(m) < 0.5, 1.0, -1.0).astype(np.float32)
    if bf16:
        X = wl.f32_to_bf16_bits(X)
        dev = torch.from_numpy(X.view(np.int16)).cuda().view(torch.bfloat16)
    else:
        dev = torch.from_numpy(X).cuda()
    Xg = api.Matrix(m, d, dense=dev)
    assert "slices=" in api.wpsgd_describe_plan(Xg, len(K_STEPS), loss)
    W = api.wpsgd_run_chains(Xg, torch.from_numpy(y).cuda(), K_STEPS, 0.5, 1e-3, loss, 9)
    ref = orc.run_chains(orc.Dense(X), y, K_STEPS, 0.5, 1e-3, loss, 9)[0]
    for i in range(len(K_STEPS)):
        assert np.linalg.norm(W[i].cpu().numpy() - ref[i]) <= TOL[loss] * max(np.linalg.norm(ref[i]), 1e-30), (d, i)
