"""Delay-SGD servers on bfloat16 rows that are no whole 16-byte pieces, and on as many samples as the per-sample kernel keeps on their
way, a few more and a few less; tolerance as in test_gpu_delay.py."""
import numpy as np
import pytest
import torch

from paper_1708_04801_amd import workloads as wl
from test_gpu_delay import compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("d", [1, 63, 511, 512 + 1, 2047, 2049, 4095, 4097])
@pytest.mark.parametrize("check", [True, False])
def test_unaligned_bf16_rows(tau, d, check):
    w = wl.delay_servers(m=97, d=d, k=10, n_lo=1, n_hi=2, tau=tau, bf16=True, spread=0.05, data_seed=tau + d)
    w.n_steps[:] = [0, 1, 2, 3, 4, 5, 7, 8, 9, 130]
    # (one column: every iterate lies along the sample, and the comparisons across it are of two zeros' rounding)
    compare(*run_both(w, tau, check=check and d > 1), f"elements tau={tau} d={d} check={check}", max_ties=2)


@pytest.mark.parametrize("d,bf16", [(1001, False), (2052, False), (1000, True)])
def test_without_delay_and_check(d, bf16):
    w = wl.delay_servers(m=97, d=d, k=10, n_lo=1, n_hi=2, tau=0, bf16=bf16, spread=0.05, data_seed=d)
    w.n_steps[:] = [0, 1, 2, 3, 4, 5, 63, 64, 65, 131]
    compare(*run_both(w, 0, check=False), f"no delay d={d}")
