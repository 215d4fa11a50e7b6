"""What users of this library have it do, as cases that can be timed and compared.

A case is one call sequence through the public entry points on one data set:

  chains     wpsgd_run_chains(_from), wpsgd_weights and wpsgd_combine: train k unequal chains and average them
  spans      wpsgd_run_spans: the periodic averaging of Deduction 2
  objective  wpsgd_objective: objective and error rate of a model on a data set
  delay      wpsgd_run_delay_chains: the delay-SGD servers of Section IV, with or without the Check function

Sizes are those of this repository's workloads, tests and benchmark, or generic ones around them.  Data are
drawn on the GPU from the seed, with the distributions that workloads.py documents.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1708_04801_amd import api

LOSS = {"hinge": api.HINGE, "logistic": api.LOGISTIC}


# Every field a case may have, with the value it takes when nothing is said.
DEFAULTS = {
    "op": "chains", "storage": "f32", "loss": "logistic", "m": 4096, "d": 64, "k": 4,
    "steps_lo": 400, "steps_hi": 1000, "steps": "uniform",     # chain lengths: uniform in [lo, hi], or lognormal (median lo, at most hi)
    "eta": 0.05, "lam": 1e-4, "shards": False, "start": 0.0,   # start: constant start vector (0: none given)
    "nnz": 80, "rows": "text",                                 # CSR: mean entries per row; text-like (Zipf columns) or binary (uniform columns)
    "spans": 1, "tau": 2, "check": True,
}


def _case(**fields):
    c = dict(DEFAULTS)
    c.update(fields)
    return c


def listed():
    return [
        # The smallest useful call: four chains on a data set that fits in cache (launches and per-step latency).
        _case(name="tiny_hinge", loss="hinge", eta=0.01, lam=1e-3),
        # A data set nobody padded: odd row length, partition-and-shuffle sampling (Algorithm 1 as written), warm start.
        _case(name="ragged_hinge", loss="hinge", m=50000, d=3001, k=100, steps_lo=500, steps_hi=3000, eta=0.01, lam=1e-3,
              shards=True, start=0.01),
        # The configuration the library's metric is quoted on: 16 KiB rows, chains that differ by up to a factor of four.
        _case(name="dense_logistic", m=262144, d=4096, k=64, steps_lo=5000, steps_hi=20000),
        # Many small unequal nodes: eight chains per compute unit.
        _case(name="many_chains", loss="hinge", m=1048576, d=256, k=2048, steps_lo=500, steps_hi=2000, eta=0.01, lam=1e-3),
        # Very wide dense rows stored in bfloat16; the largest data set.
        _case(name="wide_bf16", storage="bf16", m=65536, d=65536, k=32, steps_lo=1000, steps_hi=8000, eta=0.02, lam=1e-5),
        # Text-like sparse training: a million rows, a million features, 80 entries a row.
        _case(name="sparse_hinge", storage="csr", loss="hinge", m=1000000, d=1 << 20, k=128, steps="lognormal",
              steps_lo=10000, steps_hi=47000, eta=0.1, lam=1e-5),
        # The paper's own synthetic experiment: 5 to 10 binary features a row, eight fast nodes and two slow ones, start value 4.
        _case(name="sparse_binary", storage="csr", loss="hinge", m=460000, d=100000, k=10, steps="fast_slow",
              steps_lo=20000, steps_hi=100000, eta=1e-4, lam=0.01, nnz=8, rows="binary", start=4.0),
        # Periodic averaging: many short spans, one launch and one average each.
        _case(name="spans_logistic", op="spans", m=65536, d=1024, k=16, steps_lo=40, steps_hi=200, spans=25),
        # Evaluating a model on a dense and on a sparse data set: pure streams.
        _case(name="objective_dense", op="objective", m=262144, d=4096),
        _case(name="objective_sparse", op="objective", storage="csr", loss="hinge", m=1000000, d=1 << 20, lam=1e-5),
        # Delay-SGD servers, under the Check function and without it.
        _case(name="delay_check", op="delay", m=65536, d=4096, k=128, steps_lo=2000, steps_hi=8000, eta=0.5, lam=0.25),
        _case(name="delay_plain", op="delay", m=65536, d=4096, k=128, steps_lo=2000, steps_hi=8000, eta=0.5, lam=0.25,
              check=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["dense", "dense", "dense", "wide", "csr", "csr", "spans", "objective", "delay"])
    loss = rng.choice(["hinge", "logistic"])
    rates = {"hinge": (0.01, 1e-3), "logistic": (0.05, 1e-4)}[loss]
    if kind == "delay":
        tau = rng.randint(0, 4)
        d = rng.randint(32, 512) * 8 if rng.random() < 0.8 else rng.randint(50, 700)
        n = _log_int(rng, 200, 8000) if d % 8 == 0 else _log_int(rng, 100, 1000)
        return _case(op="delay", storage=rng.choice(["f32", "bf16"]), loss=rng.choice(["logistic", "logistic", "hinge"]),
                     m=_log_int(rng, 2000, 65536), d=d, k=_log_int(rng, 4, 200), steps_lo=max(1, n // 4), steps_hi=n, eta=0.5, lam=0.25,
                     tau=tau, check=rng.random() < 0.5)
    if kind == "csr":
        text = rng.random() < 0.6
        n = _log_int(rng, 500, 30000)
        return _case(storage="csr", loss=loss, m=_log_int(rng, 5000, 500000), d=_log_int(rng, 2000, 1 << 20), k=_log_int(rng, 2, 160),
                     steps="lognormal" if text else "uniform", steps_lo=max(1, n // 4), steps_hi=n, eta=0.1, lam=1e-5,
                     nnz=rng.randint(10, 110) if text else 8, rows="text" if text else "binary", shards=rng.random() < 0.3,
                     start=rng.choice([0.0, 0.5]))
    storage = rng.choice(["f32", "f32", "bf16"])
    if kind == "wide":                      # rows of 40 KiB and more, padded to whole 16-byte loads
        d = _log_int(rng, 12000, 65536) // 8 * 8
        n = _log_int(rng, 200, 4000)
        return _case(storage=storage, loss=loss, m=_log_int(rng, 500, 16384), d=d, k=_log_int(rng, 2, 32), steps_lo=max(1, n // 8),
                     steps_hi=n, eta=rates[0], lam=rates[1], shards=rng.random() < 0.2)
    d = _log_int(rng, 16, 8192)
    if rng.random() < 0.5:                  # half of the data sets are padded, half are not
        d = max(16, d // 8 * 8)
    m = min(_log_int(rng, 2000, 1 << 20), (1 << 29) // d)
    if kind == "objective":
        if rng.random() < 0.3:
            return _case(op="objective", storage="csr", loss=loss, m=_log_int(rng, 5000, 1000000), d=_log_int(rng, 2000, 1 << 20),
                         nnz=rng.randint(10, 110), lam=rates[1])
        return _case(op="objective", storage=storage, loss=loss, m=m, d=d, lam=rates[1])
    if kind == "spans":
        n = _log_int(rng, 20, 400)
        return _case(op="spans", storage=storage, loss=loss, m=m, d=d, k=_log_int(rng, 2, 128), steps_lo=max(1, n // 5), steps_hi=n,
                     eta=rates[0], lam=rates[1], spans=rng.randint(2, 25), shards=rng.random() < 0.3)
    k = _log_int(rng, 1, 2048)
    n = min(_log_int(rng, 100, 20000), max(100, (1 << 32) // (k * d)))
    return _case(storage=storage, loss=loss, m=m, d=d, k=min(k, m), steps_lo=max(1, n // 4), steps_hi=n, eta=rates[0], lam=rates[1],
                 shards=rng.random() < 0.3, start=rng.choice([0.0, 0.0, 0.01]))


def chain_steps(case):
    """Steps of each chain: part of the case, the same for every seed."""
    k, lo, hi = case["k"], case["steps_lo"], case["steps_hi"]
    rng = np.random.default_rng(k * 1000003 + hi)
    if case["steps"] == "lognormal":
        n = np.minimum(np.rint(rng.lognormal(math.log(lo), 0.7, size=k)), hi)
    elif case["steps"] == "fast_slow":      # eight nodes in ten have all the steps, two have the fewer
        n = np.where(np.arange(k) % 10 < 8, hi, lo)
    else:
        n = np.rint(rng.uniform(lo, hi, size=k))
        n[0] = hi                           # the longest chain has the stated length
    return n.astype(np.int64)


# ------------------------------------------------------------------------------------ data on the GPU

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _labels(case, score, gen):
    """+-1 labels: the noisy sign of the score (hinge), or drawn from a logistic model (logistic)."""
    if case["loss"] == "hinge":
        score = score + 0.1 * torch.randn(score.shape, generator=gen, device="cuda")
        return torch.where(score >= 0, 1.0, -1.0).float()
    return torch.where(torch.rand(score.shape, generator=gen, device="cuda") < torch.sigmoid(score), 1.0, -1.0).float()


def _dense(case, gen):
    """Rows N(0,1) with w* ~ N(0, 1/d) (hinge), or N(0,1)/sqrt(d) with w* ~ N(0,1) (logistic)."""
    m, d = case["m"], case["d"]
    dtype = torch.bfloat16 if case["storage"] == "bf16" else torch.float32
    unit = case["loss"] == "hinge"
    wstar = torch.randn(d, generator=gen, device="cuda") * (1.0 / math.sqrt(d) if unit else 1.0)
    X = torch.randn((m, d), generator=gen, device="cuda", dtype=dtype)
    if not unit:
        X *= 1.0 / math.sqrt(d)
    score = (X @ wstar.to(dtype)).float()
    return X, _labels(case, score, gen)


def _aligned_rows(case, gen):
    """Rows close to one direction, x = y*s*u + noise: the data on which delay-SGD servers accept updates."""
    m, d = case["m"], case["d"]
    u = torch.randn(d, generator=gen, device="cuda")
    u /= u.norm()
    y = torch.where(torch.rand(m, generator=gen, device="cuda") < 0.5, 1.0, -1.0)
    length = 0.6 + 0.4 * torch.rand(m, generator=gen, device="cuda")
    X = torch.randn((m, d), generator=gen, device="cuda")
    X *= 0.01 / math.sqrt(d)
    X.addr_(y * length, u)
    if case["storage"] == "bf16":
        X = X.to(torch.bfloat16)
    return X, y


def _csr(case, gen):
    """CSR rows with distinct ascending columns.  text: about nnz Zipf(1.1) columns, lognormal values, unit rows.
    binary: 5 to 10 uniform columns, equal values, unit rows."""
    m, d, text = case["m"], case["d"], case["rows"] == "text"
    if text:
        cdf = torch.arange(1, d + 1, device="cuda", dtype=torch.float64).pow_(-1.1).cumsum_(0)
        cdf /= cdf[-1].clone()
        cand = 2 * int(case["nnz"] + 6 * math.sqrt(case["nnz"])) + 16
        wstar = torch.randn(d, generator=gen, device="cuda") * (torch.rand(d, generator=gen, device="cuda") < 0.05)
    else:
        cand = 12
        i1 = torch.arange(1, d + 1, device="cuda")
        wstar = ((i1 % 4) * torch.where(i1 % 2 == 0, 1, -1)).float()
    lens, cols_out, vals_out, score = [], [], [], []
    for lo in range(0, m, 65536):
        r = min(65536, m - lo)
        if text:
            want = torch.poisson(torch.full((r,), float(case["nnz"]), device="cuda"), generator=gen).clamp_(1, 256).long()
            cols = torch.searchsorted(cdf, torch.rand((r, cand), generator=gen, device="cuda", dtype=torch.float64)).clamp_(max=d - 1)
        else:
            want = torch.randint(5, 11, (r,), generator=gen, device="cuda")
            cols = torch.randint(0, d, (r, cand), generator=gen, device="cuda")
        cols = cols.int().sort(dim=1).values
        prio = torch.rand((r, cand), generator=gen, device="cuda")
        prio[:, 1:][cols[:, 1:] == cols[:, :-1]] = 2.0                  # a repeated column is never kept
        cut = prio.sort(dim=1).values.gather(1, want.clamp(max=cand - 1)[:, None])
        keep = (prio < cut) & (prio < 1.5)
        n = keep.sum(dim=1)
        v = torch.randn((r, cand), generator=gen, device="cuda").exp_() if text else torch.ones((r, cand), device="cuda")
        v = torch.where(keep, v, torch.zeros_like(v))
        v /= v.norm(dim=1, keepdim=True)
        lens.append(n)
        cols_out.append(cols[keep])
        vals_out.append(v[keep])
        score.append((v * wstar[cols.long()]).sum(dim=1))
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cat(lens).cumsum(0)
    y = torch.where(torch.cat(score) >= 0, 1.0, -1.0).float()
    return row_ptr, torch.cat(cols_out), torch.cat(vals_out), y


def prepare(case, seed):
    """The data set in HBM, and the buffers a program that trains or evaluates repeatedly keeps."""
    gen = _generator(seed)
    m, d, k, loss = case["m"], case["d"], case["k"], LOSS[case["loss"]]
    if case["storage"] == "csr":
        row_ptr, col_idx, vals, y = _csr(case, gen)
        X = api.Matrix(m, d, row_ptr=row_ptr, col_idx=col_idx, vals=vals)
    else:
        dense, y = (_aligned_rows if case["op"] == "delay" else _dense)(case, gen)
        X = api.Matrix(m, d, dense=dense)
    s = {"case": dict(case), "X": X, "y": y, "seed": int(seed), "loss": loss, "n": chain_steps(case), "w_start": None}
    if case["start"]:
        s["w_start"] = torch.full((d,), float(case["start"]), device="cuda")
    if case["op"] == "objective":
        s["w"] = torch.randn(d, generator=gen, device="cuda") / math.sqrt(d)
        need = api.wpsgd_objective_workspace(X)
        s["out"] = torch.empty(2, dtype=torch.float64, device="cuda")
    elif case["op"] == "delay":
        s["w_start"] = torch.randn(d, generator=gen, device="cuda") / math.sqrt(d)
        need = api.wpsgd_run_delay_chains_workspace(X, k, case["tau"])
        s["W"] = torch.empty((k, d), dtype=torch.float32, device="cuda")
        s["accepted"] = torch.empty(k, dtype=torch.int64, device="cuda")
    elif case["op"] == "spans":
        need = api.wpsgd_run_spans_workspace(X, k, loss)
        s["w"] = torch.empty(d, dtype=torch.float32, device="cuda")
    else:
        need = api.wpsgd_run_chains_workspace(X, k, loss)
        s["W"] = torch.empty((k, d), dtype=torch.float32, device="cuda")
        s["w"] = torch.empty(d, dtype=torch.float32, device="cuda")
        s["ws_combine"] = torch.empty(max(256, api.wpsgd_combine_workspace(k, d)), dtype=torch.uint8, device="cuda")
    s["ws"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    c, X, y, n = s["case"], s["X"], s["y"], s["n"]
    if c["op"] == "objective":
        return api.wpsgd_objective(X, y, s["w"], c["lam"], s["loss"], out=s["out"], workspace=s["ws"])
    if c["op"] == "delay":
        W, accepted = api.wpsgd_run_delay_chains(X, y, n, c["eta"], c["lam"], s["loss"], s["seed"], c["tau"], check=c["check"],
                                                 w_start=s["w_start"], W=s["W"], accepted=s["accepted"], workspace=s["ws"])
        return {"W": W, "accepted": accepted}
    sampling = api.SAMPLE_SHARDS if c["shards"] else api.SAMPLE_STREAM
    if c["op"] == "spans":
        return api.wpsgd_run_spans(X, y, n, c["spans"], c["eta"], c["lam"], s["loss"], s["seed"], w_start=s["w_start"],
                                   sampling=sampling, w_out=s["w"], workspace=s["ws"])
    if c["shards"] or s["w_start"] is not None:
        W = api.wpsgd_run_chains_from(X, y, n, c["eta"], c["lam"], s["loss"], s["seed"], w_start=s["w_start"], sampling=sampling,
                                      W=s["W"], workspace=s["ws"])
    else:
        W = api.wpsgd_run_chains(X, y, n, c["eta"], c["lam"], s["loss"], s["seed"], W=s["W"], workspace=s["ws"])
    w = api.wpsgd_combine(W, api.wpsgd_weights(n, c["eta"], c["lam"]), w_out=s["w"], workspace=s["ws_combine"])
    return {"W": W, "w": w}


def work(case):
    """Each row that is visited counts once, however often it is visited; each result counts once."""
    m, d, k = case["m"], case["d"], case["k"]
    entries = {"text": case["nnz"], "binary": 7.5}[case["rows"]] if case["storage"] == "csr" else d
    row = entries * 8 + 8 if case["storage"] == "csr" else d * (2 if case["storage"] == "bf16" else 4)
    if case["op"] == "objective":
        return {"bytes": m * (row + 4) + 4 * d + 16, "flops": 2 * m * entries}
    visits = int(chain_steps(case).sum()) * case["spans"]
    rows = m * -math.expm1(-visits / m)                     # distinct rows among so many random visits
    if case["shards"]:
        rows = min(m, visits)
    # chains: w.x and the update.  delay servers: under Check x.x and a projection of every iterate kept, else one projection and the update
    per_visit = 4 * entries
    if case["op"] == "delay":
        per_visit = (2 * (max(case["tau"], 1) + 2) if case["check"] else 6) * entries
    outputs = {"chains": 4 * d * (k + 1), "spans": 4 * d, "delay": 4 * d * k + 8 * k}[case["op"]]
    return {"bytes": rows * (row + 4) + outputs, "flops": per_visit * visits}


def tolerance(case):
    """What another correct implementation of the same precision would show.  Hinge chains and delay servers carry fp64
    and round once to fp32 (two orders of summation gave equal bits); the objective stays in fp64.  Logistic chains carry
    fp32: one and two steps per reduction differ by 1.1e-7 after 20000 steps, and from fp64 by 4.2e-7 to 8e-7."""
    if case["op"] == "objective":
        return {"rel": 1e-10}
    if case["op"] == "delay" or case["loss"] == "hinge":
        return {"rel": 1e-7}
    return {"rel": 4e-6}
