"""The device-built schedule (tile table) against a re-derivation in Python: integer work, exact.

Jagged addressing must be bit-exact: every tile's rows, positions and streamed segments must be
exactly those the offsets imply, every owner row must belong to exactly one tile, tiles wholly
above the diagonal must be absent, and heavy tiles must come first.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _side(L, cp, rank):
    """Segments [(pos, len)] of one side of a sequence (rank < 0: the whole sequence)."""
    if rank < 0:
        return [(0, L)]
    c = -(-L // (2 * cp))
    segs = []
    for m in (rank, 2 * cp - 1 - rank):
        lo, hi = min(m * c, L), min((m + 1) * c, L)
        segs.append((lo, hi - lo))
    if segs[1][1] > 0 and segs[1][0] == segs[0][0] + segs[0][1]:
        segs = [(segs[0][0], segs[0][1] + segs[1][1])]
    return [s for i, s in enumerate(segs) if s[1] > 0 or i == 0]


def _expected_items(lengths, tile, causal, side, cp=1, owner_rank=-1, streamed_rank=-1):
    items = []
    obase = sbase = 0
    off = 0
    for L in lengths:
        osegs, ssegs = _side(L, cp, owner_rank), _side(L, cp, streamed_rank)
        ob = off if owner_rank < 0 else obase
        sb = off if streamed_rank < 0 else sbase
        orow = ob
        for (opos, olen) in osegs:
            for t in range(0, olen, tile):
                nrows = min(tile, olen - t)
                pos0 = opos + t
                segs, cost, srow = [], 0, sb
                for (spos, slen) in ssegs:
                    if not causal:
                        vis = slen
                    elif side == 0:
                        vis = min(max(pos0 + nrows - spos, 0), slen)
                    else:
                        vis = slen - min(max(pos0 - spos, 0), slen)
                    if vis > 0:
                        segs.append((srow, slen, spos))
                        cost += (vis + 31) // 32
                    srow += slen
                segs += [(0, 0, 0)] * (2 - len(segs))
                nseg = sum(1 for s in segs if s[1] > 0)
                items.append((orow + t, nrows, pos0, nseg, segs[0][0], segs[1][0], segs[0][1],
                              segs[1][1], segs[0][2], segs[1][2], cost, 0))
            orow += olen
        obase += sum(s[1] for s in osegs)
        sbase += sum(s[1] for s in ssegs)
        off += L
    return items


CASES = [
    ([55, 41, 33, 18], True),
    ([1, 0, 129, 128, 127, 0, 700, 3], True),
    ([300, 5, 260], False),
    (list(np.random.default_rng(5).integers(0, 600, size=70)), True),
    # batches larger than one pass of the schedule kernel's 1024 threads, kept in LDS ...
    (list(np.random.default_rng(6).integers(0, 300, size=1500)), True),
    (list(np.random.default_rng(7).integers(32, 257, size=4096)), True),
    # ... and larger than what it keeps in LDS (per-sequence bases in the workspace)
    (list(np.random.default_rng(8).integers(0, 40, size=7000)), True),
]


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("lengths,causal", CASES)
def test_full_attention_schedule(lengths, causal, side):
    import paper_2508_04711_amd as lib
    lengths = [int(x) for x in lengths]
    T = sum(lengths)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    tile = lib.hstu_schedule_tile_rows(0, 128, 128, side, T, 2, len(lengths))
    got = lib.hstu_debug_dump_schedule(off, T, 2, 128, 128, causal, 0, side, max_len=max(lengths + [1]))
    want = _expected_items(lengths, tile, causal, side)
    assert sorted(map(tuple, got.tolist())) == sorted(want)
    costs = got[:, 10].astype(np.int64)
    # Heavy tiles first, unless even the heaviest tile is small against what one of the 512
    # workgroup slots gets in total: then the library may keep the natural order.  It decides from
    # bounds (max_len for the heaviest tile, the mean length for the total), which this condition,
    # from the actual costs, implies: a cost of c means more than 32 (c - 1) streamed rows, and a
    # tile's pairs are at most 32 x tile x cost.
    if (costs.max() - 1) * 8 * 512 > costs.sum() * 2:
        assert np.all(costs[:-1] >= costs[1:]), "heavy tiles first"
    covered = np.zeros(T, dtype=np.int64)
    for it in got:
        covered[it[0]:it[0] + it[1]] += 1
    assert np.all(covered == 1), "every row in exactly one tile"


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("cp,q_rank,kv_rank", [(2, 0, 1), (2, 1, 0), (4, 3, -1), (4, 0, 0), (3, 1, 2), (1, 0, 0)])
def test_context_parallel_schedule(cp, q_rank, kv_rank, side):
    import oracle
    import paper_2508_04711_amd as lib
    lengths = [16, 5, 0, 233, 1, 400, 64, 777]
    T = sum(lengths)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    nq = len(oracle.cp_global_rows(off_np, cp, q_rank))
    nk = len(oracle.cp_global_rows(off_np, cp, kv_rank))
    tile = lib.hstu_schedule_tile_rows(0, 64, 64, side)
    got = lib.hstu_debug_dump_schedule(off, T, 2, 64, 64, True, 0, side, cp=(cp, q_rank, kv_rank, nq, nk))
    owner, streamed = (q_rank, kv_rank) if side == 0 else (kv_rank, q_rank)
    want = _expected_items(lengths, tile, True, side, cp, owner, streamed)
    assert sorted(map(tuple, got.tolist())) == sorted(want)
    covered = np.zeros(nq if side == 0 else nk, dtype=np.int64)
    for it in got:
        covered[it[0]:it[0] + it[1]] += 1
    assert np.all(covered == 1)


def test_inconsistent_offsets_never_leave_the_declared_rows():
    # offsets that overshoot the declared total: tiles are clipped to the declared rows
    import paper_2508_04711_amd as lib
    off = torch.tensor([0, 100, 5000], dtype=torch.int32, device="cuda")
    got = lib.hstu_debug_dump_schedule(off, 300, 1, 64, 64, True, 0, 0)
    for it in got:
        assert 0 <= it[0] and it[0] + it[1] <= 300
        for g in range(it[3]):
            assert 0 <= it[4 + g] and it[4 + g] + it[6 + g] <= 300


@pytest.mark.parametrize("cp", [None, (2, 1, -1)])
def test_heavy_query_tiles_are_cut_along_the_keys(cp):
    """Few query tiles, long sequences: heavy tiles appear as several items, each covering a run of
    whole 64-key tiles, which together cover the tile's visible keys exactly once."""
    import oracle
    import paper_2508_04711_amd as lib
    lengths = [9000, 5000, 700, 64]
    T = sum(lengths)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    if cp is None:
        got = lib.hstu_debug_dump_schedule(off, T, 1, 128, 128, True, 0, 0, max_len=9000)
    else:
        nq = len(oracle.cp_global_rows(off_np, cp[0], cp[1]))
        got = lib.hstu_debug_dump_schedule(off, T, 1, 128, 128, True, 0, 0,
                                           cp=(cp[0], cp[1], cp[2], nq, T), max_len=9000)
    parts = got[got[:, 11] > 0]
    whole = got[got[:, 11] == 0]
    assert len(parts) > 0, "the long sequences must produce split tiles"
    assert len(set(parts[:, 11].tolist())) == len(parts), "every part has a partial slot of its own"
    by_tile = {}
    for it in parts:
        by_tile.setdefault((int(it[0]), int(it[1]), int(it[2])), []).append(it)
    for (row0, nrows, pos0), its in by_tile.items():
        assert len(its) >= 2
        slots = sorted(int(it[11]) for it in its)
        assert slots == list(range(slots[0], slots[0] + len(its))), "consecutive slots, summed in order"
        # visible key positions of this query tile: 0 .. pos0 + nrows - 1 (causal, whole sequence streamed)
        seen = np.zeros(pos0 + nrows, dtype=np.int64)
        for it in its:
            for g in range(int(it[3])):
                spos, slen = int(it[8 + g]), int(it[6 + g])
                assert spos % 64 == 0 or cp is not None
                hi = min(spos + slen, pos0 + nrows)
                seen[spos:hi] += 1
        assert np.all(seen == 1), (row0, seen.min(), seen.max())
    # a tile is either whole or in parts, never both
    whole_tiles = {(int(it[0]), int(it[1])) for it in whole}
    assert not (whole_tiles & {(k[0], k[1]) for k in by_tile})


# ---- schedules that a wave per item builds (batches of up to 128 sequences), or that the attention kernels' waves
# work out item by item: the same items, heaviest first by their exact cost
RNG = np.random.default_rng(11)
BATCHES = [
    # one sequence per lane: up to 64, two: up to 128, the sorting builder beyond
    [int(x) for x in RNG.integers(0, 900, size=64)],
    [int(x) for x in RNG.integers(0, 900, size=65)],
    [int(x) for x in RNG.integers(0, 500, size=512)],
    [int(x) for x in RNG.integers(0, 500, size=513)],
    [0] * 63 + [4000] + [0] * 56 + [31, 32, 33, 127, 128, 129, 3990, 0],
    [int(x) for x in RNG.integers(0, 900, size=128)],
    [int(x) for x in RNG.integers(0, 900, size=129)],
    [1], [127], [128], [129],
]


def _dump(lib, lengths, heads, causal, side, cp=None, dtype=0):
    import oracle
    T = sum(lengths)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    if cp is not None:
        nq, nk = len(oracle.cp_global_rows(off_np, cp[0], cp[1])), len(oracle.cp_global_rows(off_np, cp[0], cp[2]))
        cp = cp + (nq, nk)
    got = lib.hstu_debug_dump_schedule(off, T, heads, 128, 128, causal, dtype, side, cp=cp, max_len=max(lengths + [1]))
    return got, (None if cp is None else (nq, nk))


def _heavy_first_or_large(got, heads):
    """Heavy tiles first; or, where the heaviest tile is at most half of what one of 512 workgroup slots gets, the
    order of the rows (see test_full_attention_schedule)."""
    large = (got[:, 10].max() - 1) * 2 * 512 <= got[:, 10].astype(np.int64).sum() * heads
    return bool(np.all(got[:-1, 10] >= got[1:, 10]) or large and np.all(got[:-1, 0] < got[1:, 0]))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("b", range(len(BATCHES)))
def test_items_and_exact_order_of_small_batches(b, dtype, side, causal):
    import paper_2508_04711_amd as lib
    lengths = BATCHES[b]
    got, _ = _dump(lib, lengths, 4, causal, side, dtype=dtype)
    tile = lib.hstu_schedule_tile_rows(dtype, 128, 128, side, sum(lengths), 4, len(lengths))
    assert sorted(map(tuple, got.tolist())) == sorted(_expected_items(lengths, tile, causal, side))
    assert _heavy_first_or_large(got, 4)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("cp,q_rank,kv_rank", [(4, 1, -1), (4, 0, -1), (4, 2, 2), (4, 1, 3), (8, 7, 0), (2, 1, -1), (1, 0, -1)])
@pytest.mark.parametrize("lengths", [[16, 5, 0, 233, 1, 400, 64, 777, 3000], [int(x) for x in RNG.integers(0, 1500, size=40)],
                                     [int(x) for x in RNG.integers(0, 900, size=100)],
                                     [int(x) for x in RNG.integers(0, 700, size=300)]], ids=["few", "forty", "hundred", "many"])
def test_items_and_exact_order_of_a_rank(lengths, cp, q_rank, kv_rank, side, causal):
    import paper_2508_04711_amd as lib
    got, rows = _dump(lib, lengths, 4, causal, side, cp=(cp, q_rank, kv_rank))
    owner, streamed = (q_rank, kv_rank) if side == 0 else (kv_rank, q_rank)
    want = _expected_items(lengths, 128, causal, side, cp, owner, streamed)
    assert sorted(map(tuple, got.tolist())) == sorted(want)
    assert _heavy_first_or_large(got, 4)


@pytest.mark.parametrize("cp,heads", [(None, 5), ((2, 1, -1), 3), ((4, 0, 2), 6)])
def test_query_tiles_cut_in_two(cp, heads):
    """Query tiles of few long sequences, heavy ones cut in two: a tile's two parts are neighbours in the list, cover
    what it sees, number their partial slots in order, and tiles come heaviest first."""
    import paper_2508_04711_amd as lib
    lengths = [9000, 5000, 700, 64] if cp is None else [40000, 9000, 700, 64]  # (for 512 to 1023 tiles of all heads)
    got, _ = _dump(lib, lengths, heads, True, 0, cp=cp)
    want = {(x[0], x[1], x[2]): x for x in _expected_items(lengths, 128, True, 0, *((1, -1, -1) if cp is None else cp))}
    seen, i, order, parts = set(), 0, [], 0
    while i < len(got):
        key = tuple(int(x) for x in got[i][:3])
        n = 1
        while i + n < len(got) and tuple(int(x) for x in got[i + n][:3]) == key:
            n += 1
        assert key in want and key not in seen
        seen.add(key)
        w = want[key]
        # 64 visible 32-row blocks per part at least
        assert n == (2 if w[10] >= 128 else 1), (key, n, w[10])
        rows = np.zeros(sum(lengths) + 1, dtype=np.int64)
        for k in range(n):
            it = got[i + k]
            assert int(it[11]) == (i + k + 1 if n > 1 else 0)
            for g in range(int(it[3])):
                hi = min(int(it[4 + g] + it[6 + g]), int(it[4 + g]) + max(0, key[2] + key[1] - int(it[8 + g])))
                rows[int(it[4 + g]):hi] += 1
        for g in range(w[3]):
            hi = min(w[4 + g] + w[6 + g], w[4 + g] + max(0, key[2] + key[1] - w[8 + g]))
            rows[w[4 + g]:hi] -= 1
        assert not rows.any(), key
        parts += n > 1
        order.append(w[10])
        i += n
    assert len(seen) == len(want) and parts > 0
    assert all(a >= b for a, b in zip(order, order[1:]))


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("cp", [None, (4, 1, -1), (4, 1, 2)])
@pytest.mark.parametrize("off", [[0, 100, 5000], [0, 250, 100, 280, 300], [0, -7, 90, 90, 2 ** 31 - 1], [50, 60, 10, 300]])
def test_inconsistent_offsets_of_small_batches_stay_inside(off, cp, side):
    """Offsets that overshoot, go back or start late: no item leaves the declared rows of either side."""
    import paper_2508_04711_amd as lib
    T = 300
    rows = (T, T) if cp is None else (T // 4 + 3, T if cp[2] < 0 else T // 4 + 5)
    desc = None if cp is None else cp + rows
    dev = torch.tensor(off, dtype=torch.int32, device="cuda")
    for heads in (1, 64):  # (worked out by every wave; listed by a wave per item)
        got = lib.hstu_debug_dump_schedule(dev, T, heads, 64, 64, True, 0, side, cp=desc, max_len=T)
        own, streamed = rows if side == 0 else rows[::-1]
        for it in got:
            assert 0 <= it[0] and it[0] + it[1] <= own
            for g in range(it[3]):
                assert 0 <= it[4 + g] and it[4 + g] + it[6 + g] <= streamed


def _order(lengths, heads, d, side, dtype=0):
    import paper_2508_04711_amd as lib
    off = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    got = lib.hstu_debug_dump_schedule(off, sum(lengths), heads, d, d, True, dtype, side, max_len=max(lengths))
    heavy = bool(np.all(got[:-1, 10] >= got[1:, 10]))
    rows = bool(np.all(got[:-1, 0] < got[1:, 0]))
    assert heavy != rows
    return "heavy first" if heavy else "rows"


def test_which_batches_keep_the_order_of_the_rows():
    """Few long sequences are sorted, whatever share of a slot's work their heaviest tile is (in the order of the rows
    their passes end with one sequence's tiles); many short ones are not.  fp32 lists are sorted up to the share that
    is small for any batch."""
    rng = np.random.default_rng(0)
    skewed = [int(x) for x in np.clip(np.rint(rng.lognormal(np.log(8192), 0.8, 8)), 64, 32768)]
    long12 = [int(x) for x in np.random.default_rng(3).integers(6000, 12000, size=12)]
    short = [int(x) for x in rng.integers(300, 600, size=512)]
    for d in (64, 128):
        for side in (0, 1):
            assert _order(skewed, 8, d, side) == "heavy first", (d, side)
            assert _order(long12, 8, d, side) == "heavy first", (d, side)
        assert _order(short, 4, d, 0) == "rows", d
    some = [int(x) for x in rng.integers(300, 900, size=60)]
    assert _order(some, 4, 64, 0, dtype=1) == "heavy first"
    assert _order([int(x) for x in rng.integers(100, 200, size=3000)], 4, 64, 0, dtype=1) == "rows"


@pytest.mark.parametrize("lengths,heads,cp,kv_rank,cut", [
    ([16384] * 8, 4, 4, -1, False), ([16384] * 2, 4, 4, -1, True), ([9000, 300], 1, 2, -1, True), ([16384], 2, 2, 0, True), ([2000, 1500, 900], 4, 2, 1, False)])
def test_query_tiles_of_a_partial_with_gradients(lengths, heads, cp, kv_rank, cut):
    """Side 2: what forward and dq pass in one kernel read; its tiles are cut by a rule of their own, and cut in the table
    just where the call sums partial results."""
    import oracle
    import paper_2508_04711_amd as lib
    print("dump of a partial", lengths, flush=True)
    T, r = sum(lengths), 0  # (the rank of the last positions)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    nq, nk = (len(oracle.cp_global_rows(off_np, cp, x)) for x in (r, kv_rank))
    desc = (cp, r, kv_rank, nq, nk)
    got = lib.hstu_debug_dump_schedule(off, T, heads, 128, 128, True, 0, 2, cp=desc, max_len=max(lengths))
    assert bool((got[:, 11] > 0).any()) == cut
    covered = np.zeros(nq, dtype=np.int64)
    for it in got[(got[:, 11] == 0)]:
        covered[it[0]:it[0] + it[1]] += 1
    for row0, nrows in {(int(x[0]), int(x[1])) for x in got[got[:, 11] > 0]}:
        covered[row0:row0 + nrows] += 1
    assert np.all(covered == 1)
    q, do = (torch.zeros((nq, heads, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    k, v = (torch.zeros((nk, heads, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    lib.hstu_debug_timing_begin(32)
    lib.hstu_jagged_attn_cp_partial(q, k, v, do, off, T, max(lengths), 0.1, True, cp, r, kv_rank)
    kinds = [x[0] for x in lib.hstu_debug_timing_end(32)]
    assert "fwd_dq" in kinds and ("reduce" in kinds) == cut


def _order3(lengths, heads, d):
    """The order of the key side's table as a backward call without bias builds it."""
    import paper_2508_04711_amd as lib
    off = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    got = lib.hstu_debug_dump_schedule(off, sum(lengths), heads, d, d, True, 0, 3, max_len=max(lengths))
    heavy = bool(np.all(got[:-1, 10] >= got[1:, 10]))
    assert heavy != bool(np.all(got[:-1, 0] < got[1:, 0]))
    return "heavy first" if heavy else "rows"


def test_the_key_sides_order_is_that_of_the_backward_pass(monkeypatch):
    """Where the heaviest key tile is less than a slot's share, a pass whose workgroups walk over runs keeps the order of
    the rows; at other head dimensions, with the one-wave kernel and with the bias that takes an eighth of a share."""
    from conftest import set_flags
    lengths = [512] * 96
    assert _order3(lengths, 4, 128) == "rows"
    assert _order(lengths, 4, 128, 1) == "heavy first"
    assert _order3(lengths, 4, 64) == "heavy first"
    assert _order3(lengths[:64], 4, 128) == "heavy first"
    set_flags(monkeypatch, add="DKDV_ONE_WAVE")
    assert _order3(lengths, 4, 128) == "heavy first"


@pytest.mark.parametrize("side", [2, 3])
@pytest.mark.parametrize("cp,d", [(None, 128), (None, 64), ((4, 1, -1), 128), ((4, 1, 3), 128), ((4, 1, 3), 64)])
def test_tables_of_a_call_with_gradients_hold_the_same_items(cp, d, side):
    import oracle
    import paper_2508_04711_amd as lib
    lengths = [int(x) for x in np.random.default_rng(2).integers(0, 900, size=70)]
    T = sum(lengths)
    off_np = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = torch.from_numpy(off_np).cuda()
    desc = None if cp is None else cp + tuple(len(oracle.cp_global_rows(off_np, cp[0], x)) for x in cp[1:])
    got, plain = (lib.hstu_debug_dump_schedule(off, T, 4, d, d, True, 0, s, cp=desc, max_len=900) for s in (side, side - 2))
    assert sorted(map(tuple, got.tolist())) == sorted(map(tuple, plain.tolist()))
