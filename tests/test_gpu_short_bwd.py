"""The backward pass of batches of short sequences in one kernel (max_len <= 128): groups that end one row
before, at and after a tile or a block, empty sequences (more of them in a row than a workgroup looks at at
once), a batch of one sequence, fewer groups than workgroups and more than one round of them, sequences longer
than max_len says (one, two and several tiles, on both sides of a workgroup's share), no mask, fp32 outputs.
Against the oracle; the few-terms bar where sequences are mostly shorter than a block."""
import numpy as np
import pytest
import torch

from conftest import set_flags
import oracle
import workloads
from test_gpu_parity import _check, _check_few_terms, _dev

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(17)
CASES = [
    # name, lengths, max_len, heads, d, few terms
    ("one_row", [1], 1, 1, 128, True),
    ("one_tile", [128], 128, 2, 64, False),
    ("edges", [31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 1, 127, 2, 126, 128], 128, 2, 128, False),
    ("edges", [31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 1, 127, 2, 126, 128], 128, 3, 64, False),
    ("empties", [0] * 70 + [40] + [0] * 130 + [50, 0, 0, 60, 3] + [0] * 64, 64, 2, 128, False),
    ("many", [int(x) for x in RNG.integers(0, 60, size=1500)], 60, 4, 128, True),
    ("many", [int(x) for x in RNG.integers(16, 129, size=1200)], 128, 2, 64, False),
    ("too_long", [100, 129, 20, 256, 257, 3, 700, 128, 0, 385] + [30] * 60, 128, 2, 128, False),
    ("too_long", [1000] + [5] * 200 + [300], 64, 1, 64, True),
    ("too_long_far_apart", [3] * 5 + [400] + [12] * 2300 + [129, 128, 260, 0, 0] + [7] * 700 + [500], 32, 3, 64, True),
    ("long_ones_only", [300, 129, 700, 130] + [0] * 30, 128, 2, 128, False),
    ("empties_between_shares", ([100, 27] + [0] * 300) * 30 + [0] * 5000, 128, 2, 64, False),
]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("name,lengths,max_len,H,D,few", CASES)
def test_short_backward(name, lengths, max_len, H, D, few, causal, monkeypatch):
    set_flags(monkeypatch, remove="NO_PACK", add="PACK_SHORT")
    import paper_2508_04711_amd as lib
    print("short bwd", name, H, D, causal, flush=True)
    w = workloads.custom(name, lengths, H, D, D, max_len=max_len, dtype="bf16", seed=len(lengths))
    vals = workloads.values(w)
    d = _dev(vals)
    off_np = w.seq_offsets()
    off = torch.from_numpy(off_np).cuda()
    f64 = {k: workloads.to_f64(v) for k, v in vals.items()}
    want = oracle.bwd(f64["q"], f64["k"], f64["v"], f64["d_o"], off_np, max_len, w.alpha, causal)
    for dtype in (torch.bfloat16, torch.float32):
        out = tuple(torch.full_like(d["q"], float("nan"), dtype=dtype) for _ in range(3))  # (every row is written)
        got = lib.hstu_jagged_attn_bwd(d["q"], d["k"], d["v"], d["d_o"], off, max_len, w.alpha, causal, out=out)
        if name == "too_long_far_apart":
            # The bar is a share of the RMS over rows that are sums of about as many terms: the long
            # sequences' rows (hundreds of terms, values and errors 5.5 times the others') by themselves.
            rows = np.repeat(np.array(lengths) >= 128, lengths)
            for nm, g, ref in zip(("dq", "dk", "dv"), got, want):
                _check(nm, g[torch.from_numpy(rows).cuda()], ref[rows], "bf16", name)
                _check_few_terms(nm, g[torch.from_numpy(~rows).cuda()], ref[~rows], name)
            continue
        for nm, g, ref in zip(("dq", "dk", "dv"), got, want):
            if few:
                _check_few_terms(nm, g, ref, name)
            else:
                _check(nm, g, ref, "bf16", name)


def _backward_us(lib, lengths, max_len, H, D):
    """Median time of the backward pass's kernels without their schedule, and which they are."""
    w = workloads.custom("timed", lengths, H, D, D, max_len=max_len, dtype="bf16", seed=3)
    d = _dev(workloads.values(w))
    off = torch.from_numpy(w.seq_offsets()).cuda()
    times = []
    for _ in range(9):
        lib.hstu_debug_timing_begin(16)
        lib.hstu_jagged_attn_bwd(d["q"], d["k"], d["v"], d["d_o"], off, max_len, w.alpha, True)
        torch.cuda.synchronize()
        got = [x for x in lib.hstu_debug_timing_end(16) if x[0] != "plan"]
        times.append(1e3 * sum(x[1] for x in got))
    return float(np.median(times)), {x[0] for x in got}


def test_empty_sequences_at_the_end_cost_next_to_nothing(monkeypatch):
    """(Stepped over one by one, thousands of them took 35 times as long as the batch.)"""
    set_flags(monkeypatch, remove="NO_PACK")
    import paper_2508_04711_amd as lib
    print("short bwd, trailing empties", flush=True)
    lengths = [int(x) for x in RNG.integers(16, 100, size=400)]
    plain, kinds = _backward_us(lib, lengths, 100, 4, 128)
    padded, kinds2 = _backward_us(lib, lengths + [0] * 20000, 100, 4, 128)
    assert kinds == kinds2 == {"bwd"}
    assert padded < 3 * plain + 50, (plain, padded)


def test_a_sequence_longer_than_max_len_says_is_spread_over_the_chip(monkeypatch):
    """Against the two passes over packed tiles, which take any lengths alike (629 us against 320 with the long
    sequence left to the workgroups in whose share it lies)."""
    set_flags(monkeypatch, remove="NO_PACK")
    import paper_2508_04711_amd as lib
    print("short bwd, one long sequence", flush=True)
    lengths = [int(x) for x in RNG.integers(16, 100, size=400)]
    lengths[200] = 4096
    one, kinds = _backward_us(lib, lengths, 128, 4, 128)
    set_flags(monkeypatch, add="DKDV_ONE_WAVE")
    two, kinds2 = _backward_us(lib, lengths, 128, 4, 128)
    assert kinds == {"bwd"} and kinds2 == {"dkdv", "dq"}
    assert one < 1.3 * two, (one, two)
