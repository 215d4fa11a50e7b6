"""Calls of few steps keep the kernels that start quickly.  Which kernel ran shows in the last bits of fp32 state: the
default must give those of the forced plan, and the kernel for long chains gives others."""
import math

import numpy as np
import pytest
import torch

from paper_1708_04801_amd import api
from paper_1708_04801_amd import workloads as wl

pytestmark = pytest.mark.gpu

ONE_WAVE = {"threads": 64, "block_steps": 1, "prefetch": 8}
BLOCK = {"block_steps": 16}
PIPE = {"block_steps": 16, "prefetch": 7}
OCTET = {"block_steps": 8}


def _run(d, k, n, plan, bf16=False):
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    X = (torch.randn(d, generator=g, device="cuda") + torch.randn((3000, d), generator=g, device="cuda")) / math.sqrt(d)     # (every step moves every product)
    X = X.to(torch.bfloat16) if bf16 else X
    y = torch.where(torch.rand(3000, generator=g, device="cuda") < 0.5, 1.0, -1.0)
    return api.wpsgd_run_chains(api.Matrix(3000, d, dense=X), y, np.full(k, n, dtype=np.int64), 0.5, 1e-3, wl.LOGISTIC, 9, plan=plan)


@pytest.mark.parametrize("d,k,few,enough", [
    (64, 4, 0, 1), (64, 300, 63, 64), (48, 900, 255, 256),               # at most a chain per compute unit; two; four
    (128, 4, 99, 100), (100, 300, 255, 256), (128, 900, 767, 768),
    (200, 4, 511, 512), (256, 250, 511, 512)])
def test_blocks_of_sixteen_steps(d, k, few, enough):
    blocks = PIPE if enough >= 100 and k <= 256 else BLOCK               # (long enough for the pipeline at once)
    assert torch.equal(_run(d, k, enough, None), _run(d, k, enough, blocks))
    if few:
        assert torch.equal(_run(d, k, few, None), _run(d, k, few, ONE_WAVE))
        assert not torch.equal(_run(d, k, few, blocks), _run(d, k, few, ONE_WAVE))


@pytest.mark.parametrize("d,k,few,bf16", [
    (64, 4, 31, False), (50, 256, 31, False), (64, 300, 199, False),     # at most a chain per compute unit; two
    (128, 300, 299, False), (128, 300, 255, True)])
def test_blocks_of_sixteen_steps_in_a_pipeline(d, k, few, bf16):
    assert torch.equal(_run(d, k, few + 1, None, bf16), _run(d, k, few + 1, PIPE, bf16))
    other = ONE_WAVE if bf16 else BLOCK
    assert torch.equal(_run(d, k, few, None, bf16), _run(d, k, few, other, bf16))
    assert not torch.equal(_run(d, k, few, PIPE, bf16), _run(d, k, few, other, bf16))


@pytest.mark.parametrize("d,k,few,bf16", [(1024, 4, 191, False), (513, 32, 191, False), (700, 33, 255, False), (2048, 64, 255, True)])
def test_blocks_of_eight_steps(d, k, few, bf16):
    rounds = {"helpers": -1}
    assert torch.equal(_run(d, k, few + 1, None, bf16), _run(d, k, few + 1, OCTET, bf16))
    assert torch.equal(_run(d, k, few, None, bf16), _run(d, k, few, rounds, bf16))
    assert not torch.equal(_run(d, k, few, OCTET, bf16), _run(d, k, few, rounds, bf16))


@pytest.mark.parametrize("d,slices", [(40000, 5), (16384 * 3, 6)])
def test_column_slices_of_fp32_rows(d, slices):
    """Sixteen steps and fewer: one wave per SIMD with two rounds of rows on their way; more: two waves, four rounds."""
    shallow = {"threads": 256, "slices": slices, "block_steps": 2, "prefetch": 2}
    deep = {"threads": 512, "slices": slices, "block_steps": 2, "prefetch": 4}
    assert torch.equal(_run(d, 3, 16, None), _run(d, 3, 16, shallow))
    assert torch.equal(_run(d, 3, 17, None), _run(d, 3, 17, deep))
    assert not torch.equal(_run(d, 3, 16, deep), _run(d, 3, 16, shallow))


def test_column_slices_of_bf16_rows():
    assert torch.equal(_run(12000, 3, 127, None, bf16=True), _run(12000, 3, 127, {"threads": 256, "slices": 1}, bf16=True))
    assert torch.equal(_run(12000, 3, 128, None, bf16=True), _run(12000, 3, 128, {"slices": 6}, bf16=True))


@pytest.mark.parametrize("d,k,four", [
    (65, 300, False), (129, 5000, True), (501, 5000, True), (513, 512, True), (513, 513, False), (2047, 512, True), (2049, 255, True),
    (2049, 256, False), (4093, 5000, False)])
def test_rows_that_are_not_aligned(d, k, four):
    """Four dwords at a time, or one where enough chains share the compute units."""
    flat = torch.zeros(2 * d + 1, device="cuda")
    X = api.Matrix(2, d, dense=flat[1:1 + 2 * d].view(2, d))
    plan = api.wpsgd_describe_plan(X, k, wl.HINGE)
    assert "vec=1 " in plan and ("load=4" in plan) == four, plan
