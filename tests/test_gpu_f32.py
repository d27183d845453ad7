"""The fp32 kernels at the sizes where their split can go wrong: lengths around one 32-row block, around
one block for each of a workgroup's four waves, around a 64-row step of the stream, at every head
dimension; and scores large enough that the sigmoid saturates both ways.  Bar: the stated 1e-5 x RMS."""
import pytest
import torch

import workloads
from test_gpu_parity import _run_full

pytestmark = pytest.mark.gpu

LENGTHS = [1, 31, 32, 33, 63, 0, 65, 127, 128, 129, 161, 300]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dqk,dv", [(32, 32), (64, 64), (128, 128), (128, 32), (32, 128), (64, 128)])
def test_block_edges(dqk, dv, causal):
    print("f32 edges", dqk, dv, causal, flush=True)
    w = workloads.custom("f32_edges", LENGTHS, 2, dqk, dv, max_len=300, dtype="f32", scale=1.0, seed=41)
    _run_full(w, causal=causal, backward=True)


@pytest.mark.parametrize("d", [32, 128])
def test_saturated_scores(d):
    # alpha * q.k has a standard deviation of 64: beyond +-87 the exponential's argument is clamped
    print("f32 saturated", d, flush=True)
    w = workloads.custom("f32_saturated", [200, 33], 2, d, d, max_len=200, dtype="f32", scale=8.0, seed=43)
    _run_full(w, causal=True, backward=True)
