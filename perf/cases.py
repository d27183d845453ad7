"""The work this library is used for, as a list of cases: jagged HSTU attention steps of every size,
through the public entry points of paper_2508_04711_amd as a training or serving program calls them.

A case is a dict of plain values.  "kind" says which calls a pass makes:
  fwd         hstu_jagged_attn_fwd                                   (scoring, evaluation)
  train       hstu_jagged_attn_fwd, then hstu_jagged_attn_bwd        (one attention layer of a training step)
  bias_train  the same with the timestamp bias and its table's gradient
  cp_rank     one context-parallel rank against all keys: rows into the rank's layout, partial, rows back
  cp_ring     one context-parallel rank's ring pass over the K/V parts of all ranks
Lengths are drawn from "lengths" = uniform (lo..hi) or lognormal (median exp(mu) = mid, sigma, clipped to
lo..hi) with the case's own "len_seed", so a case's work does not depend on the seed of its values.
"""
import math

import numpy as np
import torch

import paper_2508_04711_amd as hstu


def _case(name, kind, dtype, batch, lo, hi, heads, d, *, lengths="uniform", mid=0, sigma=0.0, len_seed=0, causal=True,
          cp=0, rank=0, round_to=1, buckets=0):
    return {"name": name, "kind": kind, "dtype": dtype, "batch": batch, "lo": lo, "hi": hi, "heads": heads, "d": d,
            "lengths": lengths, "mid": mid, "sigma": sigma, "len_seed": len_seed, "causal": causal, "cp": cp,
            "rank": rank, "round_to": round_to, "buckets": buckets}


def listed():
    return [
        # a handful of very short histories in fp32: the unit-test and debugging size, all latency
        _case("tiny_f32", "train", "f32", 4, 1, 64, 2, 32),
        # a training step in fp32 (reference runs, gradient checks) on a small batch of ordinary histories
        _case("train_f32", "train", "f32", 16, 64, 512, 4, 64),
        # an online scoring request: a few users, short ragged histories, forward only
        _case("score_small", "fwd", "bf16", 8, 1, 256, 4, 64),
        # a scoring batch of ordinary histories, forward only
        _case("score_batch", "fwd", "bf16", 32, 1, 1024, 4, 128),
        # a training step on ordinary long histories
        _case("train_medium", "train", "bf16", 16, 512, 4096, 4, 128),
        # the largest single-GPU training step: very skewed, very long histories
        _case("train_long", "train", "bf16", 8, 64, 32768, 8, 128, lengths="lognormal", mid=8192, sigma=0.8),
        # the same model family with the learned timestamp bias, ordinary long histories
        _case("train_bias", "bias_train", "bf16", 16, 512, 4096, 4, 128, buckets=64),
        # a large training batch of histories of a few hundred events
        _case("train_mid_batch", "train", "bf16", 1536, 300, 600, 4, 128, len_seed=7),
        # a large training batch of very short histories
        _case("train_short_batch", "train", "bf16", 8192, 16, 64, 4, 128, len_seed=7),
        # a training batch with the smaller head dimension
        _case("train_d64", "train", "bf16", 1024, 400, 800, 8, 64),
        # one context-parallel rank's share of a batch of long histories: rows in, partial, rows out
        _case("cp_rank", "cp_rank", "bf16", 8, 4096, 16384, 4, 128, cp=4, rank=1, round_to=8),
        # the same share as a ring over the K/V parts
        _case("cp_ring", "cp_ring", "bf16", 8, 4096, 16384, 4, 128, cp=4, rank=2, round_to=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# No drawn case does more than these: well inside the largest listed case's time.
_MAX_FLOPS = {"bf16": 2.5e12, "f32": 1.2e10}
_MAX_ROW_HEADS = 1.5e6


def draw(rng):
    """One more case of the ranges above: the kind first, then sizes over their logarithm."""
    while True:
        kind = rng.choice(["f32", "fwd", "fwd", "train", "train", "large", "large", "bias", "cp", "ring"])
        seed = rng.randrange(1 << 30)
        causal = rng.random() < 0.9
        if kind == "f32":
            hi = _log_int(rng, 16, 1024)
            c = _case("", "train", "f32", _log_int(rng, 2, 32), max(1, hi // rng.choice([2, 8, 64])), hi,
                      rng.choice([1, 2, 4]), rng.choice([32, 64, 128]), len_seed=seed, causal=causal)
        elif kind == "fwd":
            hi = _log_int(rng, 64, 4096)
            c = _case("", "fwd", "bf16", _log_int(rng, 1, 64), max(1, hi // rng.choice([2, 8, 64])), hi,
                      rng.choice([2, 4, 8]), rng.choice([64, 128, 128]), len_seed=seed, causal=causal)
        elif kind == "train":
            mid = _log_int(rng, 256, 8192)
            c = _case("", "train", "bf16", _log_int(rng, 4, 64), max(1, mid // 32), 4 * mid, rng.choice([2, 4, 8]),
                      rng.choice([64, 128, 128]), lengths="lognormal", mid=mid, sigma=0.8, len_seed=seed, causal=causal)
        elif kind == "large":
            hi = _log_int(rng, 24, 1024)
            c = _case("", "train", "bf16", _log_int(rng, 256, 8192), max(1, hi // rng.choice([2, 4])), hi,
                      rng.choice([2, 4, 8]), rng.choice([64, 128, 128]), len_seed=seed, causal=causal)
        elif kind == "bias":
            hi = _log_int(rng, 64, 8192)
            c = _case("", "bias_train", "bf16", _log_int(rng, 8, 512), max(1, hi // 8), hi, rng.choice([2, 4, 8]),
                      128, len_seed=seed, causal=causal, buckets=rng.choice([32, 64, 128]))
        else:
            cp = rng.choice([2, 4, 8])
            hi = _log_int(rng, 2048, 16384)
            c = _case("", "cp_rank" if kind == "cp" else "cp_ring", "bf16", _log_int(rng, 2, 16), hi // 4, hi,
                      rng.choice([2, 4, 8]), 128, len_seed=seed, cp=cp, rank=rng.randrange(cp))
        if work(c)["flops"] <= _MAX_FLOPS[c["dtype"]] and sum(_lengths(c)) * c["heads"] * c["d"] / 128 <= _MAX_ROW_HEADS:
            del c["name"]
            return c


def _lengths(case):
    rng = np.random.default_rng(case["len_seed"])
    if case["lengths"] == "lognormal":
        x = np.clip(np.rint(rng.lognormal(math.log(case["mid"]), case["sigma"], case["batch"])), case["lo"], case["hi"])
    else:
        x = rng.integers(case["lo"], case["hi"], endpoint=True, size=case["batch"])
    r = case["round_to"]
    return [int(v + r - 1) // r * r for v in x.astype(np.int64)]


def _chunks(case, rank, length):
    """The rank's two mini-chunks of one sequence as [begin, end) positions."""
    c = -(-length // (2 * case["cp"]))
    return [(min(m * c, length), min((m + 1) * c, length)) for m in (rank, 2 * case["cp"] - 1 - rank)]


def _rank_rows(case, rank):
    return sum(e - b for n in _lengths(case) for b, e in _chunks(case, rank, n))


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(1 + seed)
    lengths = _lengths(case)
    rows, heads, d = sum(lengths), case["heads"], case["d"]
    dtype, scale = (torch.bfloat16, 0.5) if case["dtype"] == "bf16" else (torch.float32, 1.0)

    def values(n=rows):
        return (torch.randn((n, heads, d), generator=gen, device="cuda") * scale).to(dtype)

    s = {"case": case, "rows": rows, "max_len": max(lengths + [1]), "alpha": 1.0 / math.sqrt(d),
         "off": torch.tensor(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), device="cuda"),
         "q": values(), "k": values(), "v": values()}
    if case["kind"] != "fwd":
        s["do"] = values()
    if case["kind"] == "bias_train":
        # sorted event times, bursts separated by idle hours; a learned table with two groups per factor of two
        rng = np.random.default_rng(seed)
        ts = [rng.integers(0, 2 ** 28) + np.cumsum(np.minimum(np.exp(rng.normal(math.log(60.0), 2.0, n)), 1e6).astype(np.int64))
              for n in lengths]
        s["ts"] = torch.tensor(np.concatenate(ts).astype(np.int32), device="cuda")
        s["table"] = torch.randn(case["buckets"], generator=gen, device="cuda")
    if case["kind"] in ("cp_rank", "cp_ring"):
        cp, rank = case["cp"], case["rank"]
        s["local"] = _rank_rows(case, rank)
        if case["kind"] == "cp_rank":
            # the layers before and after work on the global layout: outputs go back there
            s["o"], s["dq"] = torch.zeros_like(s["q"]), torch.zeros_like(s["q"])
        else:
            # a ring rank holds its own rows already; every peer holds its part of K and V
            s["q"], s["do"] = hstu.hstu_cp_reorder([s["q"], s["do"]], s["off"], rows, cp, rank, s["local"])
            parts = [hstu.hstu_cp_reorder([s["k"], s["v"]], s["off"], rows, cp, r, _rank_rows(case, r)) for r in range(cp)]
            s["k"], s["v"] = [p[0] for p in parts], [p[1] for p in parts]
            most = max(t.shape[0] for t in s["k"])
            s["recv"] = [torch.empty((most, heads, d), dtype=dtype, device="cuda") for _ in range(4)]
            s["copy_stream"] = torch.cuda.Stream()
    return s


def run(s):
    case = s["case"]
    kind, causal = case["kind"], case["causal"]
    if kind == "fwd":
        return hstu.hstu_jagged_attn_fwd(s["q"], s["k"], s["v"], s["off"], s["max_len"], s["alpha"], causal)
    if kind == "train":
        o = hstu.hstu_jagged_attn_fwd(s["q"], s["k"], s["v"], s["off"], s["max_len"], s["alpha"], causal)
        dq, dk, dv = hstu.hstu_jagged_attn_bwd(s["q"], s["k"], s["v"], s["do"], s["off"], s["max_len"], s["alpha"], causal)
        return o, dq, dk, dv
    if kind == "bias_train":
        o = hstu.hstu_jagged_attn_bias_fwd(s["q"], s["k"], s["v"], s["off"], s["ts"], s["table"], 2, s["max_len"],
                                           s["alpha"], causal)
        dq, dk, dv, dw = hstu.hstu_jagged_attn_bias_bwd(s["q"], s["k"], s["v"], s["do"], s["off"], s["ts"], s["table"], 2,
                                                        s["max_len"], s["alpha"], causal)
        return o, dq, dk, dv, dw
    cp, rank = case["cp"], case["rank"]
    if kind == "cp_rank":
        q, do = hstu.hstu_cp_reorder([s["q"], s["do"]], s["off"], s["rows"], cp, rank, s["local"])
        o, dq, dk, dv = hstu.hstu_jagged_attn_cp_partial(q, s["k"], s["v"], do, s["off"], s["rows"], s["max_len"], s["alpha"],
                                                         causal, cp, rank, -1)
        hstu.hstu_cp_reorder([o, dq], s["off"], s["rows"], cp, rank, s["local"], scatter=True, out=[s["o"], s["dq"]])
        return s["o"], s["dq"], dk, dv
    o, dq, dks, dvs = hstu.hstu_cp_ring_pass(s["q"], s["do"], s["k"], s["v"], s["off"], s["rows"], s["max_len"], s["alpha"],
                                             causal, cp, rank, recv=s["recv"], copy_stream=s["copy_stream"])
    return [o, dq] + list(dks) + list(dvs)


def work(case):
    """Visible pairs times the products' flops (4 d per pair and head forward, 10 d backward); every input
    row read once and every output row written once."""
    lengths = _lengths(case)
    rows, kind = sum(lengths), case["kind"]
    row = case["heads"] * case["d"] * (2 if case["dtype"] == "bf16" else 4)
    per_pair = (4 if kind == "fwd" else 14) * case["d"] * case["heads"]
    if kind in ("cp_rank", "cp_ring"):
        spans = [c for n in lengths for c in _chunks(case, case["rank"], n)]
        pairs = sum((e * (e + 1) - b * (b + 1)) // 2 for b, e in spans)
        local = sum(e - b for b, e in spans)
        out = row if kind == "cp_rank" else 2 * row  # the ring's outputs are fp32
        return {"bytes": 2 * local * row + 2 * rows * row + 2 * local * out + 2 * rows * out, "flops": pairs * per_pair}
    pairs = sum(n * (n + 1) // 2 if case["causal"] else n * n for n in lengths)
    tensors = 4 if kind == "fwd" else 8  # q k v -> o; q k v do -> o dq dk dv
    extra = 4 * rows + 8 * case["buckets"] if kind == "bias_train" else 0
    return {"bytes": tensors * rows * row + 4 * (len(lengths) + 1) + extra, "flops": pairs * per_pair}


def tolerance(case):
    # Measured against the same attention in 64 bits over all kinds and sizes: fp32 4.4e-7 (norm) and 6.8e-6 (largest),
    # bf16 2.4e-3 and 2.0e-2 (P and dS enter the second products as bf16, outputs are stored as bf16); about four times
    # that.
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2.5e-5}
    return {"rel": 1e-2, "max": 8e-2}
