"""A context-parallel rank's forward and dq pass in one kernel (d = 128, both outputs wanted): chunk lengths around a
block of 32 keys, a tile of 64 keys and of 128 queries, empty sequences and chunks, keys that no query sees, no mask,
outputs added to, lists that the kernels read and lists that they work out, against the oracle; tiles cut along the keys,
against the passes by themselves."""
import numpy as np
import pytest
import torch

from conftest import set_flags
import oracle
import workloads
from test_gpu_parity import _check, _check_few_terms, _dev

pytestmark = pytest.mark.gpu

# (a rank's chunk is a 2 * cp-th of a sequence)
LENGTHS = [4, 128, 0, 132, 508, 512, 516, 1, 260, 1030]
MANY = [int(x) for x in np.random.default_rng(5).integers(0, 300, size=140)]  # more than a list of one wave per item takes


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("lengths,cp,rank,kv_rank", [
    (LENGTHS, 2, 0, -1), (LENGTHS, 2, 1, -1), (LENGTHS, 4, 1, 3), (LENGTHS, 4, 3, 1), (LENGTHS, 4, 2, 2), (MANY, 2, 1, -1),
    (MANY, 2, 0, 1), ([129], 1, 0, 0)])
def test_against_the_oracle(lengths, cp, rank, kv_rank, causal):
    import paper_2508_04711_amd as lib
    print("joint", len(lengths), cp, rank, kv_rank, causal, flush=True)
    w = workloads.custom("joint", lengths, 2, 128, 128, 1030, dtype="bf16", seed=cp)
    vals = workloads.values(w)
    dev, f64 = _dev(vals), {k: workloads.to_f64(v) for k, v in vals.items()}
    off_np = w.seq_offsets()
    off, T = torch.from_numpy(off_np).cuda(), w.total_rows
    mine = oracle.cp_global_rows(off_np, cp, rank)
    keys = oracle.cp_global_rows(off_np, cp, kv_rank) if kv_rank >= 0 else np.arange(T)
    pick = lambda t, rows: t[torch.from_numpy(rows).cuda()].contiguous()
    ql, dol, kp, vp = pick(dev["q"], mine), pick(dev["d_o"], mine), pick(dev["k"], keys), pick(dev["v"], keys)
    want = oracle.cp_partial(f64["q"][mine], f64["k"][keys], f64["v"][keys], f64["d_o"][mine], off_np, w.max_len, w.alpha,
                             causal, cp, rank, kv_rank)

    def call(**kw):
        return lib.hstu_jagged_attn_cp_partial(ql, kp, vp, dol, off, T, w.max_len, w.alpha, causal, cp, rank, kv_rank, **kw)

    lib.hstu_debug_timing_begin(16)
    got = call(out_dtype=torch.float32)
    kinds = [x[0] for x in lib.hstu_debug_timing_end(16)]
    assert "fwd_dq" in kinds and "fwd" not in kinds and "dq" not in kinds
    twice = call(out=tuple(t.clone() for t in got), accumulate=True)
    rounded = call()
    for name, g, g2, gb, ref in zip(("o", "dq", "dk", "dv"), got, twice, rounded, want):
        if not np.any(ref):
            assert not torch.any(g) and not torch.any(gb), name
            continue
        _check(name, g, ref, "bf16", "joint")
        assert torch.equal(g2, g + g), name       # the same sums, added to themselves
        assert torch.equal(gb, g.bfloat16()), name


@pytest.mark.parametrize("lengths,heads,cp,kv_rank", [([9000, 300], 1, 2, -1), ([16384], 2, 2, 0), ([5000, 8200, 64], 2, 1, 0)])
def test_cut_tiles(lengths, heads, cp, kv_rank, monkeypatch):
    """Few workgroups and long sequences: tiles are cut along the keys and both outputs' parts summed."""
    import paper_2508_04711_amd as lib
    print("joint cut", lengths, heads, flush=True)
    T, r = sum(lengths), cp - 1
    gen = torch.Generator(device="cuda").manual_seed(3)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    nq = len(oracle.cp_global_rows(off_np, cp, r))
    nk = len(oracle.cp_global_rows(off_np, cp, kv_rank)) if kv_rank >= 0 else T
    val = lambda n: (torch.randn((n, heads, 128), generator=gen, device="cuda") * 0.5).bfloat16()
    q, do, k, v = val(nq), val(nq), val(nk), val(nk)

    def call():
        lib.hstu_debug_timing_begin(32)
        res = lib.hstu_jagged_attn_cp_partial(q, k, v, do, off, T, max(lengths), 128 ** -0.5, True, cp, r, kv_rank,
                                              out_dtype=torch.float32)
        return res, [x[0] for x in lib.hstu_debug_timing_end(32)]

    got, kinds = call()
    assert "fwd_dq" in kinds and "reduce" in kinds
    set_flags(monkeypatch, add="DKDV_ONE_WAVE")  # (keeps the passes apart)
    set_flags(monkeypatch, add="NO_SPLIT")
    want, kinds = call()
    assert "fwd_dq" not in kinds and "reduce" not in kinds
    # the same products of the same operands; sums of up to 16384 fp32 terms in another order (1e-5 of the largest), and a
    # dS whose last bits differ may round to the neighbouring bf16 operand, 2^-8 of one term of thousands
    for name, a, b in zip(("o", "dq", "dk", "dv"), got, want):
        assert (a - b).abs().max().item() <= 2e-4 * b.abs().max().item(), name


@pytest.mark.parametrize("flag", ["DKDV_ONE_WAVE", "FWD_TILE_128", "FWD_TILE_256"])
def test_passes_kept_apart(flag, monkeypatch):
    """The flags that keep a partial's forward and dq pass apart: its o is the forward-only partial's, bit for bit."""
    import paper_2508_04711_amd as lib
    print("joint apart", flag, flush=True)
    set_flags(monkeypatch, add=flag)
    lengths, heads, cp, r = [5000, 300, 0, 129], 2, 2, 1
    T = sum(lengths)
    gen = torch.Generator(device="cuda").manual_seed(4)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    nq = len(oracle.cp_global_rows(off_np, cp, r))
    val = lambda n: (torch.randn((n, heads, 128), generator=gen, device="cuda") * 0.5).bfloat16()
    q, do, k, v = val(nq), val(nq), val(T), val(T)

    def call(d_o):
        lib.hstu_debug_timing_begin(32)
        res = lib.hstu_jagged_attn_cp_partial(q, k, v, d_o, off, T, max(lengths), 128 ** -0.5, True, cp, r, -1,
                                              out_dtype=torch.float32)
        return res[0], [x[0] for x in lib.hstu_debug_timing_end(32)]

    (with_gradients, kinds), (alone, _) = call(do), call(None)
    assert "fwd" in kinds and "dq" in kinds and "fwd_dq" not in kinds
    assert torch.equal(with_gradients, alone)


@pytest.mark.parametrize("batch,length,q_rank,kv_rank,causal,max_len,joint", [
    (50, 64, 1, -1, True, 256, True), (60, 99, 1, -1, True, 256, False), (60, 101, 1, -1, True, 256, True), (120, 101, 1, -1, True, 256, False),
    (60, 108, 0, 1, True, 256, False), (60, 112, 0, 1, True, 256, True), (60, 312, 1, 0, True, 256, False), (60, 324, 1, 0, True, 256, True),
    (60, 196, 1, 1, True, 256, False), (60, 204, 1, 1, True, 256, True), (60, 78, 0, -1, False, 256, False), (60, 80, 0, -1, False, 256, True),
    (130, 198, 1, -1, True, 256, False), (130, 201, 1, -1, True, 256, True),
    (60, 99, 1, -1, True, 704, False), (60, 99, 1, -1, True, 736, True), (60, 100, 1, 0, True, 1503, True)])
def test_many_short_sequences(batch, length, q_rank, kv_rank, causal, max_len, joint):
    """Both sides of the lines below which the passes of many short sequences are apart (streamed rows of a sequence by the
    workgroups that rows and batch allow for) and of the longest sequence that max_len allows for, two ranks, 8 heads."""
    import paper_2508_04711_amd as lib
    print("joint short", batch, length, q_rank, kv_rank, causal, flush=True)
    lengths = [length + (i % 3) - 1 for i in range(batch)]
    lengths[-1] += length * batch - sum(lengths)
    w = workloads.custom("joint_short", lengths, 8, 128, 128, max_len, dtype="bf16", seed=batch + length)
    vals = workloads.values(w)
    dev, f64 = _dev(vals), {k: workloads.to_f64(v) for k, v in vals.items()}
    off_np = w.seq_offsets()
    off, T = torch.from_numpy(off_np).cuda(), w.total_rows
    mine = oracle.cp_global_rows(off_np, 2, q_rank)
    keys = oracle.cp_global_rows(off_np, 2, kv_rank) if kv_rank >= 0 else np.arange(T)
    pick = lambda t, rows: t[torch.from_numpy(rows).cuda()].contiguous()
    lib.hstu_debug_timing_begin(16)
    got = lib.hstu_jagged_attn_cp_partial(pick(dev["q"], mine), pick(dev["k"], keys), pick(dev["v"], keys), pick(dev["d_o"], mine),
                                          off, T, w.max_len, w.alpha, causal, 2, q_rank, kv_rank, out_dtype=torch.float32)
    kinds = [x[0] for x in lib.hstu_debug_timing_end(16)]
    assert ("fwd_dq" in kinds) == joint and ("fwd" in kinds) == ("dq" in kinds) == (not joint)
    want = oracle.cp_partial(f64["q"][mine], f64["k"][keys], f64["v"][keys], f64["d_o"][mine], off_np, w.max_len, w.alpha,
                             causal, 2, q_rank, kv_rank)
    for name, g, ref in zip(("o", "dq", "dk", "dv"), got, want):
        _check_few_terms(name, g, ref, "joint")
