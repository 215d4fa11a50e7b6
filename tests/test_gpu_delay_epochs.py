"""What a team of workgroups on one delay-SGD server does at the ends of its epochs, on streams whose acceptances are chosen by position.

Two kinds of rows: short ones, on which the hinge does not fire and whose update, a decay, the Check function accepts, and long
ones, on which eta*lambda + eta*|x|^2 >= 1 and nothing but a server's very first update passes (a decay as well).  Short rows are those
that the stream names at the chosen positions and nowhere else."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

D, M, ETA, LAM = 64, 1 << 20, 0.5, 0.04
LONG, SHORT = np.zeros(D, dtype=np.float32), np.zeros(D, dtype=np.float32)
LONG[0] = 10.0
SHORT[:2] = 1.1 * np.cos(0.1), 1.1 * np.sin(0.1)          # (not along the iterates: across it they get shorter)
START = np.zeros(D, dtype=np.float32)
START[0] = 1000.0                                          # 1000 * 1.1 * 0.98^270 > 1: the hinge stays silent


def _problem(rows):
    X = torch.from_numpy(LONG).cuda().repeat(M, 1)
    X[torch.from_numpy(rows).cuda()] = torch.from_numpy(SHORT).cuda()
    return api.Matrix(M, D, dense=X), torch.ones(M, device="cuda"), torch.from_numpy(START).cuda()


def _oracle(idx, rows):
    kinds = np.isin(idx, rows).astype(np.int64)
    W, accepted, _ = orc.delay_sgd(orc.Dense(np.stack([LONG, SHORT])), np.ones(2, dtype=np.float32), kinds, ETA, LAM, wl.HINGE, 1,
                                   w0=START.astype(np.float64), check=True)
    return W, accepted


def test_a_record_of_256_epochs_before_is_not_believed():
    """Epochs are told apart by eight bits.  The second of two members sees the other's acceptance at place 0 in one epoch (in its own batches,
    places 4 to 7, 12 to 15 and so on, there is none), accepts in its own first batch in the next 255, and in the one after finds nothing
    before its second batch, at place 13."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    k, n = units // 2, 9400
    at, base = [7000], 7001                       # (acceptances this late that the owner keeps its team)
    for place in [0] + [7] * 255 + [13]:
        at.append(base + place)
        base = at[-1] + 1
    for seed in range(400):
        idx = api.wpsgd_sample_indices(seed, 0, 0, n, M)
        rows = np.unique(idx[at])
        if np.isin(idx, rows).sum() == len(at):
            break
    else:
        pytest.fail("no such stream")
    X, y, start = _problem(rows)
    want_w, want = _oracle(idx, rows)
    assert want == len(at) + 1
    W, accepted = api.wpsgd_run_delay_chains(X, y, np.full(k, n, dtype=np.int64), ETA, LAM, wl.HINGE, seed, 1, w_start=start)
    assert int(accepted[0]) == want
    assert np.linalg.norm(W[0].cpu().numpy() - want_w) <= 1e-6 * np.linalg.norm(want_w)


def test_epochs_that_end_without_an_acceptance():
    """An epoch has 2^22 samples at most; the acceptances here are the first sample, a few behind the end of the epoch that begins soon
    after and a few about the end of the next."""
    epoch = 1 << 22
    n = 2 * epoch + 5000
    idx = api.wpsgd_sample_indices(3, 0, 0, n, M)
    seen = np.bincount(idx, minlength=M)
    once = np.flatnonzero(seen[idx] == 1)          # (a good eight visits a row: one position in 3000)
    late = once[once >= 100 + epoch]
    rows = idx[np.concatenate([late[:2], late[-2:]])]
    assert late[0] < 1 + 2 * epoch
    X, y, start = _problem(rows)
    want_w, want = _oracle(idx, rows)
    assert want == 5
    W, accepted = api.wpsgd_run_delay_chains(X, y, np.array([n, 10], dtype=np.int64), ETA, LAM, wl.HINGE, 3, 1, w_start=start)
    assert accepted.tolist() == [want, 1]
    assert np.linalg.norm(W[0].cpu().numpy() - want_w) <= 1e-6 * np.linalg.norm(want_w)


@pytest.mark.parametrize("n", [385, 700])
@pytest.mark.parametrize("at", [[], [1, 2, 3], [5, 9, 13, 14, 90], list(range(1, 30)), list(range(1, 34)), list(range(1, 60)), list(range(0, 700, 32)),
                                list(range(3, 700, 23)), list(range(3, 700, 25)), list(range(35, 700, 3)), list(range(100, 300)), list(range(1, 700)),
                                [380, 381, 384]])
def test_teams_that_dissolve(n, at):
    """Acceptances that come thick from the first, from somewhere on, for a while or at the very end: the owner sends its team away, or keeps it."""
    at = [0] + [p for p in at if 0 < p < n]
    for seed in range(2000):
        idx = api.wpsgd_sample_indices(seed, 0, 0, n, M)
        rows = np.unique(idx[at])
        if np.isin(idx, rows).sum() == len(at):
            break
    else:
        pytest.fail("no such stream")
    X, y, start = _problem(rows)
    want_w, want = _oracle(idx, rows)
    for others in (0, 20):
        steps = np.full(1 + others, n, dtype=np.int64)
        W, accepted = api.wpsgd_run_delay_chains(X, y, steps, ETA, LAM, wl.HINGE, seed, 1, w_start=start)
        assert int(accepted[0]) == want
        assert np.linalg.norm(W[0].cpu().numpy() - want_w) <= 1e-6 * np.linalg.norm(want_w)


@pytest.mark.parametrize("share", [1.0, 0.5, 0.2, 0.1, 0.05, 0.02, 0.005])
@pytest.mark.parametrize("n", [385, 1100, 3000])
@pytest.mark.parametrize("k", [1, 7, 60, 128])
def test_any_share_of_acceptances(share, n, k):
    """Teams that begin, end at once, dissolve or never begin: the bits of a call whose servers outnumber the compute units (no teams)."""
    m = 4096
    kinds = torch.from_numpy((np.random.default_rng(n + k).random(m) < share)[:, None]).cuda()
    X = api.Matrix(m, D, dense=torch.where(kinds, torch.from_numpy(SHORT).cuda(), torch.from_numpy(LONG).cuda()).contiguous())
    y, start = torch.ones(m, device="cuda"), torch.from_numpy(START).cuda() * 1e25
    steps = np.random.default_rng(k).integers(n // 2, n + 1, k).astype(np.int64)
    steps[0] = n
    units = torch.cuda.get_device_properties(0).multi_processor_count
    W0, acc0 = api.wpsgd_run_delay_chains(X, y, np.concatenate([steps, np.ones(units, dtype=np.int64)]), ETA, LAM, wl.HINGE, 5, 1, w_start=start)
    W1, acc1 = api.wpsgd_run_delay_chains(X, y, steps, ETA, LAM, wl.HINGE, 5, 1, w_start=start)
    assert torch.equal(acc0[:k], acc1)
    assert torch.equal(W0[:k].view(torch.int32), W1.view(torch.int32))
    assert int(acc1[0]) >= share * n / 2
