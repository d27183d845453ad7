"""The one-block-at-a-time kernels of d = 64 (launches of more than 2048 workgroups): sequences that end at, one row
before and one row after a block and a tile, empty ones and long ones among them, a sorted schedule and one in natural
order, packed tiles, no mask, fp32 outputs, head counts with and without an XCD-aware map.  Against the oracle."""
import numpy as np
import pytest
import torch

from conftest import set_flags
import oracle
import workloads
from test_gpu_bias import _run as _run_bias
from test_gpu_parity import _check_few_terms, _dev

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(23)
EDGES = [31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 0, 255, 256, 257, 1]
CASES = [
    # name, lengths, heads, packed
    ("sorted", EDGES * 8 + [700, 1, 1500], 8, False),
    ("natural", [int(x) for x in RNG.integers(129, 400, size=600)], 2, False),
    ("three_heads", EDGES * 24, 3, False),
    ("packed", [int(x) for x in RNG.integers(0, 300, size=900)] + EDGES, 4, True),
]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("name,lengths,H,packed", CASES)
def test_many_workgroups(name, lengths, H, packed, causal, monkeypatch):
    if packed:
        set_flags(monkeypatch, remove="NO_PACK", add="PACK_SHORT")
    else:
        set_flags(monkeypatch, add="NO_PACK")
    import paper_2508_04711_amd as lib
    tiles = sum(lengths) // 128 + (0 if packed else len(lengths)) + 1  # (the bound the launch is sized from)
    assert tiles * H > 2048
    print("lean", name, H, causal, flush=True)
    w = workloads.custom(name, lengths, H, 64, 64, max_len=max(lengths), dtype="bf16", seed=len(lengths))
    vals = workloads.values(w)
    d = _dev(vals)
    off_np = w.seq_offsets()
    off = torch.from_numpy(off_np).cuda()
    f64 = {k: workloads.to_f64(v) for k, v in vals.items()}
    want_o = oracle.fwd(f64["q"], f64["k"], f64["v"], off_np, w.max_len, w.alpha, causal)
    want = oracle.bwd(f64["q"], f64["k"], f64["v"], f64["d_o"], off_np, w.max_len, w.alpha, causal)
    for dtype in (torch.bfloat16, torch.float32):
        out = [torch.full_like(d["q"], float("nan"), dtype=dtype) for _ in range(4)]  # (every row is written)
        lib.hstu_jagged_attn_fwd(d["q"], d["k"], d["v"], off, w.max_len, w.alpha, causal, out=out[0])
        lib.hstu_jagged_attn_bwd(d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, causal, out=tuple(out[1:]))
        for nm, g, ref in zip(("o", "dq", "dk", "dv"), out, (want_o,) + tuple(want)):
            # The last keys and the first queries of every sequence are sums of one term or a few, and with
            # 8 M elements some such are over 7 RMS: an operand's rounding (2^-9 of a term) and the output's own
            # (2^-9) are then 2.7e-2 RMS, more than the many-terms bar gives.
            _check_few_terms(nm, g, ref, name)


@pytest.mark.parametrize("repeat,H,many", [(2, 4, False), (18, 8, True)])
@pytest.mark.parametrize("dqk,dv,bias", [(64, 32, False), (32, 128, False), (32, 64, False), (32, 32, True), (128, 64, False), (32, 32, False)])
def test_forms_on_both_sides_of_the_limit(dqk, dv, bias, repeat, H, many, monkeypatch):
    """The other head dimensions whose masks have a form for few workgroups and one for many (dq pass, and the forward pass at
    32 / 64, 32 / 128, 128 / 64 and 32 / 32)."""
    set_flags(monkeypatch, add="NO_PACK")
    lengths = EDGES * repeat
    assert ((sum(lengths) // 128 + len(lengths) + 1) * H > 2048) == many
    print("lean", dqk, dv, bias, many, flush=True)
    w = workloads.custom("lean_dims", lengths, H, dqk, dv, max_len=257, dtype="bf16", seed=dqk + dv)
    if bias:
        _run_bias(w, "events", nb=40, f=2, seed=3, check=_check_few_terms)
        return
    import paper_2508_04711_amd as lib
    vals = workloads.values(w)
    d = _dev(vals)
    off_np = w.seq_offsets()
    off = torch.from_numpy(off_np).cuda()
    f64 = {k: workloads.to_f64(v) for k, v in vals.items()}
    want = (oracle.fwd(f64["q"], f64["k"], f64["v"], off_np, w.max_len, w.alpha, True),) + tuple(
        oracle.bwd(f64["q"], f64["k"], f64["v"], f64["d_o"], off_np, w.max_len, w.alpha, True))
    got = (lib.hstu_jagged_attn_fwd(d["q"], d["k"], d["v"], off, w.max_len, w.alpha, True),) + tuple(
        lib.hstu_jagged_attn_bwd(d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, True))
    for nm, g, ref in zip(("o", "dq", "dk", "dv"), got, want):
        _check_few_terms(nm, g, ref, "lean")
