"""The kernel that decides delay-SGD samples one at a time: calls under the Check function whose servers are too brief for a table of
row quantities, on rows of 16-byte pieces and of single elements, and calls with more servers than compute units.  Tolerance as in
test_gpu_delay.py."""
import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl
from test_gpu_delay import compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("d,bf16", [(64, False), (2048, False), (2052, False), (4096, False), (64, True), (2048, True), (2056, True), (4096, True),
                                    (1001, False), (1001, True)])
def test_brief_servers_under_check(tau, d, bf16):
    """Fewer than 96 samples each, less than a quarter as many as there are rows: no table."""
    w = wl.delay_servers(m=1600, d=d, k=8, n_lo=1, n_hi=2, tau=tau, bf16=bf16, data_seed=300 + tau + d)
    w.n_steps[:] = [95, 0, 1, 3, 4, 5, 64, 93]
    assert 4 * w.n_steps.sum() < w.m
    Wg, acc_g, Wo, acc_o, gap = run_both(w, tau, check=True)
    compare(Wg, acc_g, Wo, acc_o, gap, f"brief tau={tau} d={d}", max_ties=1)
    assert acc_o.max() >= 3


@pytest.mark.parametrize("check", [False, True])
def test_more_servers_than_compute_units(check):
    w = wl.delay_servers(m=400, d=129, k=1100, n_lo=1, n_hi=40, tau=0, data_seed=4)
    compare(*run_both(w, 0, check=check), f"many check={check}", max_ties=8)


def test_two_servers_share_a_compute_unit():
    """Twice as many servers as compute units, side by side: a unit that holds one at a time needs twice as long (measured 1.9; side by side
    1.3; 1.65 lies between)."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    w = wl.delay_servers(m=2000, d=2047, k=2 * units, n_lo=400, n_hi=401, tau=4, data_seed=6)
    w.n_steps[:] = 400
    X, y = api.matrix_from_workload(w), torch.from_numpy(w.y).cuda()
    start = torch.from_numpy(w.meta["w_start"]).cuda()
    space = torch.empty(api.wpsgd_run_delay_chains_workspace(X, w.k, 4), dtype=torch.uint8, device="cuda")

    def time(k):
        took = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            api.wpsgd_run_delay_chains(X, y, w.n_steps[:k], w.eta, w.lam, w.loss, w.seed, 4, w_start=start, workspace=space)
            b.record()
            torch.cuda.synchronize()
            took.append(a.elapsed_time(b))
        return min(took[1:])

    one, two = time(units), time(2 * units)
    print(f"{units} servers {one * 1e3:.0f} us, {2 * units} servers {two * 1e3:.0f} us")
    assert two < 1.65 * one
