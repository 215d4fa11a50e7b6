"""Delay-SGD servers under the Check function that together visit few of many rows: what the test needs of a row is kept per visit, the
servers' visits one server after the other.  Tolerance as in test_gpu_delay.py."""
import time

import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl
from test_gpu_delay import compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 3, 63, 64, 65, 70, 129, 300, 4097])
@pytest.mark.parametrize("n", [97, 380, 800])
def test_servers_find_their_visits(k, n):
    """With teams and without (fewer than 384 samples, more servers than compute units), idle servers at the ends and in between."""
    n = n if k <= 300 else 97
    rng = np.random.default_rng(k + n)
    steps = rng.integers(0, 12 if k > 100 else n + 1, k).astype(np.int64)
    steps[rng.integers(0, k, max(1, k // 5))] = 0
    steps[k // 2] = n
    m = int(4 * steps.sum()) + 5
    w = wl.delay_servers(m=m, d=64, k=k, n_lo=1, n_hi=2, tau=1, spread=0.05, data_seed=k)
    w.n_steps[:] = steps
    Wg, acc_g, Wo, acc_o, gap = run_both(w, 1, check=True)
    compare(Wg, acc_g, Wo, acc_o, gap, f"visits k={k} n={n}", max_ties=max(1, k // 100))
    assert acc_o.max() >= 3


def test_many_servers_cost_what_their_visits_cost():
    """Every visit looks up whose it is.  Servers of ten samples: eight times as many took 33 times as long where every visit added up
    the servers before its own, and take 6 times as long; 16 lies between."""
    m, d = 1 << 22, 64
    X = api.Matrix(m, d, dense=torch.randn((m, d), device="cuda") * 0.1)
    y = torch.ones(m, device="cuda")

    def clock(k):
        n = np.full(k, 10, dtype=np.int64)
        n[0] = 100
        space = torch.empty(api.wpsgd_run_delay_chains_workspace(X, k, 1), dtype=torch.uint8, device="cuda")
        took = []
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            api.wpsgd_run_delay_chains(X, y, n, 0.05, 0.1, wl.LOGISTIC, 1, 1, workspace=space)
            torch.cuda.synchronize()
            took.append(time.perf_counter() - t)
        return min(took[1:])

    few, many = clock(5000), clock(40000)
    print(f"5000 servers {few * 1e6:.0f} us, 40000 servers {many * 1e6:.0f} us")
    assert many < 16 * few


@pytest.mark.parametrize("k", [1, 10])
@pytest.mark.parametrize("d", [60, 64, 72])
def test_short_rows_keep_their_teams(k, d):
    """The least room for the teams' tables.  Servers of 4000 samples in teams take a tenth of the time that they take in a call whose servers
    outnumber the compute units (no teams); a half lies between."""
    m = 1 << 18
    X = api.Matrix(m, d, dense=torch.randn((m, d), device="cuda") * 0.05)
    y = torch.ones(m, device="cuda")
    units = torch.cuda.get_device_properties(0).multi_processor_count

    def clock(n):
        space = torch.empty(api.wpsgd_run_delay_chains_workspace(X, len(n), 1), dtype=torch.uint8, device="cuda")
        took = []
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            api.wpsgd_run_delay_chains(X, y, n, 0.05, 0.1, wl.LOGISTIC, 1, 1, workspace=space)
            torch.cuda.synchronize()
            took.append(time.perf_counter() - t)
        return min(took[1:])

    n = np.full(k, 4000, dtype=np.int64)
    teams, alone = clock(n), clock(np.concatenate([n, np.ones(units, dtype=np.int64)]))
    print(f"teams {teams * 1e6:.0f} us, alone {alone * 1e6:.0f} us")
    assert teams < 0.5 * alone
