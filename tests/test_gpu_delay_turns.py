"""Delay-SGD calls with teams of workgroups on several streams and from several host threads: launches that do not fit on the device
together run one after the other.  Results bit for bit as on one stream."""
import threading
import time

import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu


class Calls:
    def __init__(self, k, n, streams, d=1024):
        w = wl.delay_servers(m=4096, d=d, k=k, n_lo=n // 4, n_hi=n, tau=2, data_seed=8)
        w.n_steps[0] = n
        self.w, self.X, self.y = w, api.matrix_from_workload(w), torch.from_numpy(w.y).cuda()
        self.start = torch.from_numpy(w.meta["w_start"]).cuda()
        need = api.wpsgd_run_delay_chains_workspace(self.X, k, 2)
        self.streams = [torch.cuda.Stream() for _ in range(streams)]
        self.spaces = [torch.empty(need, dtype=torch.uint8, device="cuda") for _ in range(streams)]
        torch.cuda.synchronize()

    def __call__(self, i):
        with torch.cuda.stream(self.streams[i]):
            return api.wpsgd_run_delay_chains(self.X, self.y, self.w.n_steps, self.w.eta, self.w.lam, self.w.loss, self.w.seed, 2,
                                              w_start=self.start, workspace=self.spaces[i])


def _same(got, want):
    return torch.equal(got[1], want[1]) and torch.equal(got[0].view(torch.int32), want[0].view(torch.int32))


@pytest.mark.parametrize("k,n", [(3, 3000), (40, 2000), (128, 1500), (200, 1000)])
def test_many_streams(k, n):
    """More streams than the latest launches that are kept in mind."""
    calls = Calls(k, n, 11, d=256)
    want = calls(0)
    torch.cuda.synchronize()
    got = [calls(i) for _ in range(2) for i in range(11)]
    torch.cuda.synchronize()
    assert all(_same(g, want) for g in got)


def test_several_host_threads():
    calls = Calls(128, 1500, 4, d=256)
    want = calls(0)
    torch.cuda.synchronize()
    got = [[] for _ in range(4)]

    def work(i):
        for _ in range(6):
            got[i].append(calls(i))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert all(len(g) == 6 for g in got) and all(_same(x, want) for g in got for x in g)


@pytest.mark.parametrize("k,n", [(2, 6000), (4, 6000), (60, 3000), (128, 1500)])
def test_units_taken_by_another_call(k, n):
    """Teams some of whose members, or all but the owner, start late: a call without the Check function, which is not put in turn, holds the compute
    units and gives them back a few at a time."""
    calls = Calls(k, n, 2)
    want = calls(0)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    space = torch.empty(api.wpsgd_run_delay_chains_workspace(calls.X, 2 * units, 2), dtype=torch.uint8, device="cuda")
    other = torch.cuda.Stream()
    for shape in (np.linspace(50, 4000, 2 * units), np.where(np.arange(2 * units) % 3, 300, 3000), np.where(np.arange(2 * units) < 100, 100, 2000)):
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            api.wpsgd_run_delay_chains(calls.X, calls.y, shape.astype(np.int64), calls.w.eta, calls.w.lam, calls.w.loss, calls.w.seed, 2, check=False,
                                       w_start=calls.start, workspace=space)
        got = [calls(1) for _ in range(3)]
        torch.cuda.synchronize()
        assert all(_same(g, want) for g in got)


def test_two_streams_take_no_longer_than_one_after_the_other():
    """Half as many servers as compute units.  128 servers: one call 824 us, two on two streams 1565 us in turn; 2045 us where the second's
    servers find their teams' units taken (2.5 times one call; 2.3 lies between)."""
    calls = Calls(torch.cuda.get_device_properties(0).multi_processor_count // 2, 4000, 2)

    def clock(which):
        took = []
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for i in which:
                calls(i)
            torch.cuda.synchronize()
            took.append(time.perf_counter() - t)
        return float(np.median(took[1:]))

    one, two = clock([0]), clock([0, 1])
    print(f"one call {one * 1e6:.0f} us, two {two * 1e6:.0f} us")
    assert two < 2.3 * one
