"""The fp32 kernels at the sizes where their split can go wrong: lengths around one 32-row block, around
one block for each of a workgroup's four waves, around a 64-row step of the stream, at every head
dimension; scores large enough that the sigmoid saturates both ways, and scores over the whole range of fp32.
Bar: the stated 1e-5 x RMS, or 1e-6 of the value where a result has one term."""
import numpy as np
import pytest
import torch

import oracle
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


@pytest.mark.parametrize("d,heads,batch,one", [(32, 4, 191, True), (32, 4, 192, False), (64, 4, 191, True),
                                               (128, 2, 31, True), (128, 2, 32, False), (64, 3, 1, True)])
def test_both_passes_in_one_launch(d, heads, batch, one):
    """The backward pass on both sides of the limits up to which it is one launch (counted in the workgroups that
    rows and batch allow for: 1536, and 128 at d = 128), and with a number of them that is no multiple of eight."""
    import paper_2508_04711_amd as lib
    print("f32 one launch", d, heads, batch, flush=True)
    lengths = [32 + (i % 3) - 1 for i in range(batch)]
    lengths[-1] += 32 * batch - sum(lengths)
    w = workloads.custom("f32_one", lengths, heads, d, d, max_len=64, dtype="f32", scale=1.0, seed=47)
    _run_full(w, causal=True, backward=True)
    t = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    lib.hstu_debug_timing_begin(16)
    lib.hstu_jagged_attn_bwd(t["q"], t["k"], t["v"], t["d_o"], off, w.max_len, w.alpha, True)
    kinds = [x[0] for x in lib.hstu_debug_timing_end(16) if x[0] != "plan"]
    assert kinds == (["bwd"] if one else ["dkdv", "dq"])


@pytest.mark.parametrize("d,batch,max_len,one", [(64, 74, 1025, True), (64, 75, 1025, False), (64, 75, 1024, True),
                                                 (32, 75, 1025, True)])
def test_one_launch_of_long_sequences(d, batch, max_len, one):
    """d = 64 and a max_len beyond 1024: one launch up to 600 workgroups that rows and batch allow for, 4 heads."""
    import paper_2508_04711_amd as lib
    print("f32 one launch, long", d, batch, max_len, flush=True)
    w = workloads.custom("f32_one_long", [32] * batch, 4, d, d, max_len=max_len, dtype="f32", scale=1.0, seed=48)
    _run_full(w, causal=True, backward=True)
    t = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    lib.hstu_debug_timing_begin(16)
    lib.hstu_jagged_attn_bwd(t["q"], t["k"], t["v"], t["d_o"], off, w.max_len, w.alpha, True)
    kinds = [x[0] for x in lib.hstu_debug_timing_end(16) if x[0] != "plan"]
    assert kinds == (["bwd"] if one else ["dkdv", "dq"])


@pytest.mark.parametrize("d", [32, 128])
def test_saturated_scores(d):
    # alpha * q.k has a standard deviation of 64: many scores lie beyond what the exponential resolves
    print("f32 saturated", d, flush=True)
    w = workloads.custom("f32_saturated", [200, 33], 2, d, d, max_len=200, dtype="f32", scale=8.0, seed=43)
    _run_full(w, causal=True, backward=True)


# x = alpha * q.k of one pair: silu(x) is x above ~17 and 0 below ~-104, to the end of fp32's range
EXTREME = [-3.4e38, -3e37, -1e30, -1e6, -120.0, -104.5, -103.0, -30.0, -1.0, 0.0, 1.0, 30.0, 88.5, 103.0, 1e6, 1e30, 3e37,
           2.5e38, 3.4e38]


def _silu64(x):
    """silu and its derivative in 64 bits; the sigmoid of the far negative side without overflow."""
    z = np.exp(-np.abs(x))
    sg = np.where(x >= 0, 1.0, z) / (1.0 + z)
    return x * sg, sg * (1.0 + x * (1.0 - sg))


@pytest.mark.parametrize("d", [32, 128])
def test_scores_over_the_whole_range(d):
    """Sequences of one row: one pair each, so every output is one term."""
    import paper_2508_04711_amd as lib
    print("f32 extreme scores", d, flush=True)
    x = np.array(EXTREME, dtype=np.float32)
    n = len(x)
    zero = lambda: torch.zeros((n, 1, d), dtype=torch.float32, device="cuda")
    q, k, v, do = zero(), zero(), zero(), zero()
    qs = np.where(np.abs(x) > 1e6, np.float32(1e19), np.float32(1))
    ks = (x / qs).astype(np.float32)
    q[:, 0, 0], k[:, 0, 0] = torch.from_numpy(qs).cuda(), torch.from_numpy(ks).cuda()
    v[:, 0, 1], do[:, 0, 1] = 0.5, 0.25
    off = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    o = lib.hstu_jagged_attn_fwd(q, k, v, off, 1, 1.0, True)
    dq, dk, dv = lib.hstu_jagged_attn_bwd(q, k, v, do, off, 1, 1.0, True)
    xx = (qs * ks).astype(np.float64)  # the product as fp32 rounds it
    p, dp = _silu64(xx)
    ds = 0.125 * dp
    # a term below fp32's smallest normal number may be flushed to zero
    for name, got, want in (("o", o[:, 0, 1], p * 0.5), ("dv", dv[:, 0, 1], p * 0.25), ("dq", dq[:, 0, 0], ds * ks),
                            ("dk", dk[:, 0, 0], ds * qs)):
        g = got.double().cpu().numpy()
        bad = np.abs(g - want) > 1e-6 * np.abs(want) + 1e-35
        assert not bad.any(), (name, x[bad], g[bad], want[bad])


def test_table_entries_at_the_ends_of_the_range():
    """A timestamp table whose entries are fp32's lowest value (a mask), its highest and infinity."""
    import paper_2508_04711_amd as lib
    print("f32 extreme table", flush=True)
    big = float(np.finfo(np.float32).max)
    ts = torch.tensor([0, 0, 2, 4, 8], dtype=torch.int32, device="cuda")
    off = torch.tensor([0, 2, 5], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k = [torch.randn((5, 1, 32), generator=g, device="cuda") for _ in range(2)]
    v = torch.full((5, 1, 32), 1e-3, device="cuda")
    alpha = 32 ** -0.5

    def want(bias):  # o of row 4 from its pairs with rows 2, 3, 4
        s = (q[4, 0].double() @ k[2:5, 0].double().T).cpu().numpy() + np.array(bias)
        return float(np.sum(_silu64(alpha * s)[0]) * 1e-3)

    def last(tab):
        return float(lib.hstu_jagged_attn_bias_fwd(q, k, v, off, ts, tab, 0, 1, alpha, True)[4, 0, 0])
    # differences 6, 4, 0 of the last row's pairs: buckets 2, 2, 0
    masked = torch.tensor([0.25, 0.5, -big], dtype=torch.float32, device="cuda")
    assert abs(last(masked) - want([-big, -big, 0.25])) <= 1e-5 * abs(want([-big, -big, 0.25])) + 1e-9
    high = torch.tensor([0.25, 0.5, big / 4], dtype=torch.float32, device="cuda")
    assert abs(last(high) / want([big / 4, big / 4, 0.25]) - 1) <= 1e-5
    assert last(torch.tensor([0.25, 0.5, float("inf")], dtype=torch.float32, device="cuda")) == float("inf")


def _short_list_bytes(rows, batch, passes):
    """Room for one list of 64-row items per pass: per item the 64-byte record, its place in the order, an entry of
    the (unused) table of cut tiles, 8 bytes per streamed tile; four arrays of an entry per sequence; alignment."""
    items = rows // 64 + batch + 1
    return passes * (items * (64 + 4 + 16 + 8) + 4 * 4 * (batch + 1) + 64 + 8 * 64 + 256) + 4096


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dqk,dv", [(32, 32), (128, 128), (64, 128)])
@pytest.mark.parametrize("lengths", [LENGTHS, [40, 64, 1] * 300])
def test_a_workspace_for_64_row_items_is_enough(lengths, dqk, dv, causal):
    """The query names the room for lists of 32-row items; with less than that the lists are of 64-row items, each
    shared by two workgroups, and the results are the same bits."""
    import paper_2508_04711_amd as lib
    print("f32 short list", len(lengths), dqk, dv, causal, flush=True)
    w = workloads.custom("f32_short_list", lengths, 3, dqk, dv, max_len=300, dtype="f32", scale=1.0, seed=47)
    d = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    ws = lambda passes: torch.empty(_short_list_bytes(w.total_rows, w.batch, passes), dtype=torch.uint8, device="cuda")
    a = (d["q"], d["k"], d["v"])
    o = [lib.hstu_jagged_attn_fwd(*a, off, 300, w.alpha, causal, workspace=x) for x in (None, ws(1))]
    assert torch.equal(o[0], o[1])
    g = [lib.hstu_jagged_attn_bwd(*a, d["d_o"], off, 300, w.alpha, causal, workspace=x) for x in (None, ws(2))]
    for x, y in zip(*g):
        assert torch.equal(x, y)
    with pytest.raises(lib.HstuError) as e:
        small = torch.empty((w.total_rows // 64) * 84, dtype=torch.uint8, device="cuda")
        lib.hstu_jagged_attn_fwd(*a, off, 300, w.alpha, causal, workspace=small)
    assert e.value.status == -4


def test_long_sequences_with_the_short_list():
    """Rows enough that only the short list fits, with more than one head per tile and a sorted schedule."""
    import paper_2508_04711_amd as lib
    lengths = [int(x) for x in np.random.default_rng(3).integers(1, 2000, size=70)]
    w = workloads.custom("f32_short_long", lengths, 2, 32, 32, max_len=2000, dtype="f32", scale=1.0, seed=48)
    d = {k: v.cuda() for k, v in workloads.values(w).items()}
    off = torch.from_numpy(w.seq_offsets()).cuda()
    need = lib.hstu_jagged_attn_workspace_bytes((w.batch, 2, 32, 32, 2000, 1.0, True, 1, w.total_rows), 1)
    small = _short_list_bytes(w.total_rows, w.batch, 2)
    assert small < need
    args = (d["q"], d["k"], d["v"], d["d_o"], off, 2000, w.alpha, True)
    want = lib.hstu_jagged_attn_bwd(*args)
    got = lib.hstu_jagged_attn_bwd(*args, workspace=torch.empty(small, dtype=torch.uint8, device="cuda"))
    for x, y in zip(want, got):
        assert torch.equal(x, y)


def test_forward_without_a_workspace_takes_seven_million_rows():
    """The static array holds the 64-row list of 1000 sequences with 7 M rows."""
    import paper_2508_04711_amd as lib
    print("f32 static", flush=True)
    off = torch.linspace(0, 7_000_000, 1001, device="cuda").round().to(torch.int32)
    off[:997] = torch.arange(997, device="cuda", dtype=torch.int32) * 40  # (short ones, so that this is no long run)
    off[997:1000] = torch.tensor([40000, 41000, 42000], dtype=torch.int32, device="cuda")
    off[1000] = 43000
    q = torch.randn((7_000_000, 1, 32), dtype=torch.float32, device="cuda")
    out = torch.full_like(q, 7.0)
    lib.hstu_jagged_attn_fwd_static(q, q, q, off, 1000, 0.1, True, out)
    want = lib.hstu_jagged_attn_fwd(q, q, q, off, 1000, 0.1, True, out=torch.full_like(q, 7.0))
    assert torch.equal(out, want) and bool((out[43000:] == 7.0).all())


@pytest.mark.parametrize("dqk,dv,heads", [(128, 128, (1 << 18) + 3), (32, 128, (1 << 18) + 1), (32, 32, (1 << 20) + 5)])
def test_rows_of_more_than_128_megabytes(dqk, dv, heads):
    """Heads enough that a block of rows reaches beyond 32-bit offsets; a few of them against 64 bits."""
    import paper_2508_04711_amd as lib
    print("f32 wide rows", dqk, dv, heads, flush=True)
    lengths = [5, 1, 34]
    T = sum(lengths)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k = [torch.randn((T, heads, dqk), generator=g, device="cuda") for _ in range(2)]
    v, do = [torch.randn((T, heads, dv), generator=g, device="cuda") for _ in range(2)]
    alpha = dqk ** -0.5
    o = lib.hstu_jagged_attn_fwd(q, k, v, off, 7, alpha, True)
    dq, dk, dv_ = lib.hstu_jagged_attn_bwd(q, k, v, do, off, 7, alpha, True)
    for h in (0, 1, heads // 2, heads - 1):
        f = [x[:, h].double().cpu().numpy()[:, None] for x in (q, k, v, do)]
        off_np = off.cpu().numpy()
        want = (oracle.fwd(f[0], f[1], f[2], off_np, 7, alpha, True),) + tuple(oracle.bwd(*f, off_np, 7, alpha, True))
        for name, got, ref in zip(("o", "dq", "dk", "dv"), (o, dq, dk, dv_), want):
            err = np.abs(got[:, h].double().cpu().numpy() - ref[:, 0]).max() / np.sqrt(np.mean(ref ** 2))
            assert err <= 1e-5, (name, h, err)


@pytest.mark.parametrize("d,scale,bound", [(128, 1.0, 2.42e-7), (64, 1.0, 3.2e-7), (32, 1.0, 3.3e-7), (64, 3.0, 3.8e-7),
                                           (64, 8.0, 4.1e-7)])
def test_error_against_64_bits(d, scale, bound):
    """The 2-norm of each output's error over the output's, at most what sums taken key by key in fp32, with the
    precise exponential and IEEE division, were off for the same inputs (the bound; the largest of the four outputs)."""
    import paper_2508_04711_amd as lib
    lengths = {128: [200, 129, 33], 32: [40, 64, 3, 500]}.get(d, [300, 1, 77, 512, 64] if scale == 1.0 else [300, 100])
    print("f32 error", d, scale, flush=True)
    w = workloads.custom("e", lengths, 2, d, d, max_len=max(lengths), dtype="f32", scale=scale, seed=9)
    vals = workloads.values(w)
    x = {k: v.cuda() for k, v in vals.items()}
    f = {k: workloads.to_f64(v) for k, v in vals.items()}
    off_np = w.seq_offsets()
    off = torch.from_numpy(off_np).cuda()
    want = (oracle.fwd(f["q"], f["k"], f["v"], off_np, w.max_len, w.alpha, True),) + tuple(
        oracle.bwd(f["q"], f["k"], f["v"], f["d_o"], off_np, w.max_len, w.alpha, True))
    got = (lib.hstu_jagged_attn_fwd(x["q"], x["k"], x["v"], off, w.max_len, w.alpha, True),) + tuple(
        lib.hstu_jagged_attn_bwd(x["q"], x["k"], x["v"], x["d_o"], off, w.max_len, w.alpha, True))
    for name, g, ref in zip(("o", "dq", "dk", "dv"), got, want):
        err = np.linalg.norm(g.double().cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= bound, (name, err)
