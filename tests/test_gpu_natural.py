"""Schedules in natural order built by many workgroups: batches that end one sequence before, at and after a
workgroup's 64, empty sequences, offsets that end before the declared rows, head counts with and without an
XCD-aware map, no mask.  Against the oracle."""
import numpy as np
import pytest
import torch

from conftest import set_flags
import oracle
import workloads
from test_gpu_parity import _check_few_terms, _dev

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(41)


def _lengths(n, lo, hi, empties=0):
    x = [int(v) for v in RNG.integers(lo, hi, size=n)]
    for i in range(empties):
        x[(i * 7) % n] = 0
    return x


CASES = [
    # name, lengths, heads, d
    ("b191", _lengths(191, 260, 300), 8, 64),
    ("b192", _lengths(192, 260, 300), 8, 128),
    ("b193", _lengths(193, 260, 300, 30), 8, 128),
    ("b449", _lengths(449, 200, 400), 3, 64),
]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("name,lengths,H,D", CASES)
def test_natural_order(name, lengths, H, D, causal, monkeypatch):
    set_flags(monkeypatch, add="NO_PACK")
    import paper_2508_04711_amd as lib
    print("natural", name, H, D, causal, flush=True)
    w = workloads.custom(name, lengths, H, D, D, max_len=max(lengths), dtype="bf16", seed=len(lengths))
    # (the rule: the heaviest item is less than half of what one of 512 workgroup slots gets)
    mean = w.total_rows // w.batch
    assert 128 * w.max_len * 2 < mean * mean // (2 if causal else 1) * w.batch // 512 * H
    vals = workloads.values(w)
    d = _dev(vals)
    off_np = w.seq_offsets()
    off = torch.from_numpy(off_np).cuda()
    f64 = {k: workloads.to_f64(v) for k, v in vals.items()}
    want_o = oracle.fwd(f64["q"], f64["k"], f64["v"], off_np, w.max_len, w.alpha, causal)
    want = oracle.bwd(f64["q"], f64["k"], f64["v"], f64["d_o"], off_np, w.max_len, w.alpha, causal)
    out = [torch.full_like(d["q"], float("nan")) for _ in range(4)]  # (every row is written)
    lib.hstu_jagged_attn_fwd(d["q"], d["k"], d["v"], off, w.max_len, w.alpha, causal, out=out[0])
    lib.hstu_jagged_attn_bwd(d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, causal, out=tuple(out[1:]))
    for nm, g, ref in zip(("o", "dq", "dk", "dv"), out, (want_o,) + tuple(want)):
        _check_few_terms(nm, g, ref, name)


def test_offsets_that_end_before_the_declared_rows(monkeypatch):
    """Rows beyond the last offset belong to no sequence: the outputs there stay as they were."""
    set_flags(monkeypatch, add="NO_PACK")
    import paper_2508_04711_amd as lib
    lengths = _lengths(300, 200, 300)
    w = workloads.custom("short_offsets", lengths, 4, 64, 64, max_len=300, dtype="bf16", seed=3)
    d = _dev(workloads.values(w))
    off = torch.from_numpy(w.seq_offsets()).cuda()
    cut = off.clone()
    end = int(off[270])
    cut[270:] = end
    full = lib.hstu_jagged_attn_fwd(d["q"], d["k"], d["v"], off, 300, w.alpha, True)
    out = torch.full_like(full, 7.0)
    lib.hstu_jagged_attn_fwd(d["q"], d["k"], d["v"], cut, 300, w.alpha, True, out=out)
    assert torch.equal(out[:end], full[:end])
    assert bool((out[end:] == 7.0).all())
