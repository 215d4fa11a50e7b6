"""Delay-SGD servers under the Check function on several workgroups each, against the fp64 oracle and against one
workgroup per server.

A team decides with the same sums in the same order as a server alone, so its results are compared bit for bit with
those of the same call on so many servers that none has a team; tolerance against the oracle as in test_gpu_delay.py."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl
from test_gpu_delay import compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("d,bf16", [(64, False), (2048, False), (2052, False), (4096, False), (2056, True)])
@pytest.mark.parametrize("m", [64, 1500, 40000])
def test_teams_against_the_oracle(tau, d, bf16, m):
    """Lengths about the shortest that has a team, servers that stay alone beside them, an idle one; rows visited often (a table
    per row) and seldom (a table per visit)."""
    w = wl.delay_servers(m=min(m, 4000 if d > 2000 else m), d=d, k=6, n_lo=300, n_hi=900, tau=tau, bf16=bf16, data_seed=3 * tau + d)
    w.n_steps[:] = [385, 0, 1, 1030, 31, 33]
    compare(*run_both(w, tau, check=True), f"team tau={tau} d={d}", max_ties=1)


@pytest.mark.parametrize("n", [383, 384, 385, 2047, 2049])
@pytest.mark.parametrize("k", [1, 2, 127, 129, 250])
def test_teams_change_nothing(n, k):
    """The first servers of a call with more servers than compute units (nobody has a team) and the same servers in a
    call of their own: equal counts and equal bits."""
    w = wl.delay_servers(m=700, d=256, k=k, n_lo=1, n_hi=2, tau=2, data_seed=n)
    rng = np.random.default_rng(n + k)
    lengths = rng.integers(1, n + 1, k)
    lengths[0] = n
    X, y = api.matrix_from_workload(w), torch.from_numpy(w.y).cuda()
    start = torch.from_numpy(w.meta["w_start"]).cuda()

    def run(lengths):
        W, accepted = api.wpsgd_run_delay_chains(X, y, lengths.astype(np.int64), w.eta, w.lam, w.loss, w.seed, 2, w_start=start)
        return W[:k].cpu().numpy(), accepted[:k].cpu().numpy()

    units = torch.cuda.get_device_properties(0).multi_processor_count
    W0, acc0 = run(np.concatenate([lengths, np.ones(units, dtype=np.int64)]))
    W1, acc1 = run(lengths)
    assert acc1.tolist() == acc0.tolist()
    assert np.array_equal(W1.view(np.uint32), W0.view(np.uint32))


@pytest.mark.parametrize("n", [420, 900])
def test_many_acceptances_dissolve_a_team(n):
    """Rows on which the hinge does not fire and a start vector far out along them: every update is a decay, which the Check
    function accepts, sample after sample, until the hinge fires (0.98^j * 100 * 1.1 < 1) or the stream ends."""
    rng = np.random.default_rng(n)
    u = np.zeros(512, dtype=np.float32)
    u[:] = 1.0 / np.sqrt(512.0)
    X = (1.1 * u + 1e-3 * rng.standard_normal((300, 512))).astype(np.float32)
    w = wl.delay_servers(m=300, d=512, k=3, n_lo=n, n_hi=n + 1, tau=1, loss=wl.HINGE, data_seed=1)
    w.dense[:], w.y[:] = X, 1.0
    w.meta["w_start"] = 100.0 * u
    w.lam = 0.04
    Wg, acc_g, Wo, acc_o, gap = run_both(w, 1, check=True)
    compare(Wg, acc_g, Wo, acc_o, gap, "decay", max_ties=0)
    assert acc_o.min() > 150


def test_teams_on_two_streams_and_again():
    """Two calls at once, which together want more workgroups than the device seats, several times over: a team is whoever
    is running, and the results do not depend on it."""
    w = wl.delay_servers(m=2000, d=4096, k=40, n_lo=600, n_hi=2000, tau=2, data_seed=5)
    X, y = api.matrix_from_workload(w), torch.from_numpy(w.y).cuda()
    start = torch.from_numpy(w.meta["w_start"]).cuda()
    n = w.n_steps.astype(np.int64)
    want = api.wpsgd_run_delay_chains(X, y, n, w.eta, w.lam, w.loss, w.seed, 2, w_start=start)
    torch.cuda.synchronize()
    need = api.wpsgd_run_delay_chains_workspace(X, w.k, 2)
    streams = [torch.cuda.Stream() for _ in range(2)]
    spaces = [torch.empty(need, dtype=torch.uint8, device="cuda") for _ in streams]
    out = []
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        for s, space in zip(streams, spaces):
            with torch.cuda.stream(s):
                out.append(api.wpsgd_run_delay_chains(X, y, n, w.eta, w.lam, w.loss, w.seed, 2, w_start=start, workspace=space))
    torch.cuda.synchronize()
    for W, accepted in out:
        assert torch.equal(accepted, want[1])
        assert torch.equal(W.view(torch.int32), want[0].view(torch.int32))
