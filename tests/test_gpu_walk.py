"""The walking dk/dv kernel with two waves per 32 keys (d = 128, large batches and packed tiles, bf16 outputs):
items of one, two and three 32-row blocks (shorter ones are padded to three), a single item, fewer items than
workgroups, more items than one round of workgroups, tiles that end one row after or before a block, no mask,
head counts with and without an XCD-aware map.  Against the oracle (bf16 outputs: the stated bar plus their own
rounding; the few-terms bar where sequences are mostly shorter than a block)."""
import numpy as np
import pytest
import torch

from conftest import set_flags
import oracle
import workloads
from test_gpu_parity import _check, _check_few_terms, _dev

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(91)
# (max_len, the normaliser, is more than 128 throughout: below, packed tiles take the backward pass in one kernel)
CASES = [
    # name, lengths, heads, few terms
    ("one_row", [1], 1, True),
    ("one_tile", [128], 2, False),
    ("block_edges", [31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 161], 2, False),
    ("three_heads", [200, 0, 7, 255, 256, 1], 3, False),
    ("one_long", [1000], 4, False),
    ("many_short", [int(x) for x in RNG.integers(0, 24, size=700)], 8, True),
    ("many_items", [int(x) for x in RNG.integers(60, 200, size=300)], 4, False),
]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("name,lengths,H,few", CASES)
def test_walking_dkdv(name, lengths, H, few, causal, monkeypatch):
    set_flags(monkeypatch, remove="NO_PACK", add="PACK_SHORT")
    import paper_2508_04711_amd as lib
    print("walk", name, H, causal, flush=True)
    w = workloads.custom(name, lengths, H, 128, 128, max_len=max(max(lengths), 129), dtype="bf16", seed=len(lengths))
    vals = workloads.values(w)
    d = _dev(vals)
    off_np = w.seq_offsets()
    off = torch.from_numpy(off_np).cuda()
    f64 = {k: workloads.to_f64(v) for k, v in vals.items()}
    want = oracle.bwd(f64["q"], f64["k"], f64["v"], f64["d_o"], off_np, w.max_len, w.alpha, causal)
    out = [torch.full_like(d["q"], float("nan")) for _ in range(3)]  # (every row is written)
    lib.hstu_debug_timing_begin(16)
    got = lib.hstu_jagged_attn_bwd(d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, causal, out=tuple(out))
    assert [x[0] for x in lib.hstu_debug_timing_end(16)] == ["plan", "dkdv", "dq"]
    for nm, g, ref in zip(("dq", "dk", "dv"), got, want):
        if few:
            _check_few_terms(nm, g, ref, name)
        else:
            _check(nm, g, ref, "bf16", name)


@pytest.mark.parametrize("causal", [True, False])
def test_walking_dkdv_over_a_large_batch_in_natural_order(causal, monkeypatch):
    """Per-sequence tiles in natural order (mean length above the packed tiles' limit), against the
    one-wave kernel, which the other tests hold against the oracle: the same products with the same operand
    roundings, so the two differ by their fp32 sums' order and one rounding to bf16."""
    set_flags(monkeypatch, remove="NO_PACK")
    import paper_2508_04711_amd as lib
    lengths = [int(x) for x in np.random.default_rng(5).integers(129, 520, size=1400)]
    w = workloads.custom("natural", lengths, 4, 128, 128, max_len=520, dtype="bf16", seed=6)
    # (the rule: the heaviest item is less than an eighth of what one of 512 workgroup slots gets)
    mean = w.total_rows // w.batch
    assert 128 * w.max_len * 8 < mean * mean // (2 if causal else 1) * w.batch // 512 * 4
    print("walk natural", causal, flush=True)
    d = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    args = (d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, causal)
    _, dk, dv = lib.hstu_jagged_attn_bwd(*args)
    set_flags(monkeypatch, add="DKDV_ONE_WAVE")
    _, dk1, dv1 = lib.hstu_jagged_attn_bwd(*args)
    for a, b in ((dk, dk1), (dv, dv1)):
        # two neighbouring bf16 values are 2^-7 of the value apart at most; sums of up to 520 terms in
        # another order differ by up to 520 * 2^-24 of the terms' magnitudes, of the order of the RMS
        a, b = a.float(), b.float()
        rms = b.pow(2).mean().sqrt()
        excess = (a - b).abs() - (2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 520 * 2.0 ** -24 * rms)
        assert excess.max().item() <= 0, excess.max().item()


RUNS = [
    # name, lengths, heads: sorted ascending and descending, with empty sequences and tiles of one row, few items a run
    ("ascending", sorted(int(x) for x in RNG.integers(1, 700, size=700)), 4),
    ("descending", sorted((int(x) for x in RNG.integers(1, 900, size=401)), reverse=True), 8),
    ("empty_ones", [int(x) for x in RNG.integers(200, 420, size=450) * RNG.integers(0, 2, size=450)], 8),
    ("one_row_tiles", [129, 257, 385] * 301, 2),
    ("one_head", [int(x) for x in RNG.integers(100, 260, size=1701)], 1),
    ("few", [512] * 96, 4),
]


def _walked(lib, *args, **kw):
    """The backward pass's gradients and the form of its dk/dv kernel."""
    lib.hstu_debug_timing_begin(16)
    got = lib.hstu_jagged_attn_bwd(*args, **kw)
    return got, [x[0] for x in lib.hstu_debug_timing_end(16) if x[0] != "plan"][0]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("name,lengths,H", RUNS)
def test_runs_of_equal_work(name, lengths, H, causal, monkeypatch):
    """Per-sequence tiles in natural order from where the heaviest item is less than a slot's share (1 of 512) on, the
    workgroups walking runs of equal work, against the one-wave kernel within the bound of the test above; every
    row is written."""
    set_flags(monkeypatch, add="NO_PACK")  # (two of the batches have a mean below the packed tiles' limit)
    import paper_2508_04711_amd as lib
    longest = max(lengths)
    w = workloads.custom(name, lengths, H, 128, 128, max_len=longest, dtype="bf16", seed=8)
    mean = w.total_rows // w.batch
    assert 128 * longest < mean * mean // (2 if causal else 1) * w.batch // 512 * H
    print("runs", name, causal, flush=True)
    d = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    args = (d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, causal)
    out = tuple(torch.full_like(d["q"], float("nan")) for _ in range(3))
    (_, dk, dv), form = _walked(lib, *args, out=out)
    assert form == "dkdv_runs"
    set_flags(monkeypatch, add="DKDV_ONE_WAVE")
    (_, dk1, dv1), form = _walked(lib, *args)
    assert form == "dkdv"
    for a, b in ((dk, dk1), (dv, dv1)):
        a, b = a.float(), b.float()
        rms = b.pow(2).mean().sqrt()
        excess = (a - b).abs() - (2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + longest * 2.0 ** -24 * rms)
        assert excess.max().item() <= 0, excess.max().item()  # (NaN fails too)


@pytest.mark.parametrize("lengths,H,form", [
    ([512] * 96, 4, "dkdv_runs"), ([512] * 64, 4, "dkdv"), ([512] * 96, 3, "dkdv"), ([256] * 500, 4, "dkdv")])
def test_which_batches_are_walked_in_runs(lengths, H, form):
    """(The last: packed tiles, whose walk has no runs of equal work.)"""
    import paper_2508_04711_amd as lib
    w = workloads.custom("which", lengths, H, 128, 128, max_len=512, dtype="bf16", seed=9)
    d = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    _, got = _walked(lib, d["q"], d["k"], d["v"], d["d_o"], off, w.max_len, w.alpha, True)
    assert got == form


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("name,lengths,H", RUNS)
def test_work_before_every_item(name, lengths, H, causal, monkeypatch):
    """What the runs are taken from: each item's record holds the work of all items before it, the header all of it (an
    item's 32-row blocks, three at least, and three more), with sequences without rows in between."""
    set_flags(monkeypatch, add="NO_PACK")
    import paper_2508_04711_amd as lib
    T = sum(lengths)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    nbytes = lib.hstu_jagged_attn_workspace_bytes((len(lengths), H, 128, 128, max(lengths), 1.0, causal, 0, T), 0)
    ws = torch.zeros((nbytes + 63) // 64 * 64, dtype=torch.uint8, device="cuda")
    items = lib.hstu_debug_dump_schedule(off, T, H, 128, 128, causal, 0, 3, max_len=max(lengths), workspace=ws)
    assert np.all(items[:-1, 0] < items[1:, 0]), "the order of the rows"
    records = ws.view(torch.int32).reshape(-1, 16).cpu().numpy()  # (an item is a 64-byte record; the header is the first)
    first = [i for i in range(len(records) - len(items) + 1)
             if np.array_equal(records[i, :4], items[0, :4]) and np.array_equal(records[i:i + len(items), :4], items[:, :4])]
    assert len(first) == 1
    streamed = items[:, 6] - (items[:, 2] if causal else 0)  # rows of the sequence at or after the tile's first key
    work = np.maximum(3, (streamed + 31) // 32) + 3
    assert np.array_equal(records[first[0]:first[0] + len(items), 14], np.cumsum(work) - work)
    assert records[0, 3] == work.sum()
