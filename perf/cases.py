"""Performance cases of the forward pass: what a serving program asks of this library.

Every case is a forward of one model through `RecModel.forward`,
`RecModel.forward_static` or a pipelined model's `forward` ... `drain`, on
inputs that sit in device memory already.  Shapes are those of the workloads in
`paper_2203_07424_amd/synth.py` (Table I's DLRM-RMC1/2/3 and MT-WnD rows) and
batch sizes from a single query to the largest fused batch of the batch-size
sweep in `bench.py`.  Tables, ids, dense features and weights are drawn on the
device from the seed alone, with the distributions of `synth.py`: rows
U(-0.05, 0.05), ids Zipf over scattered ranks or uniform, lengths fixed or
Poisson clamped to [1, 200], dense N(0, 1), weights and biases N(0, 1/fan_in).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2203_07424_amd import binding


def _case(name, tables, rows, dim, dtype, batch, dense, length, bottom, hidden, lengths="fixed",
          ids="uniform", alpha=0.0, interaction="dot", towers=1, mode="forward", batches=1,
          stream_rows=False):
    """bottom: widths behind the dense input ("" = no Bottom-FC); hidden: Predict-FC
    widths between its input and the one logit per tower ("" = none)."""
    c = dict(tables=tables, rows=rows, dim=dim, dtype=dtype, batch=batch, dense=dense, length=length,
             lengths=lengths, ids=ids, alpha=alpha, bottom=bottom, hidden=hidden,
             interaction=interaction, towers=towers, mode=mode, batches=batches, stream_rows=stream_rows)
    if name:
        c["name"] = name
    return c


# The models of synth.py as keyword sets; batch sizes are the cases' own.
_TINY = dict(tables=8, rows=100_000, dim=32, dtype="f32", dense=13, length=20, bottom="256-128-32", hidden="64")
_RMC1 = dict(tables=10, rows=4_000_000, dim=64, dtype="f32", dense=256, length=80, ids="zipf", alpha=1.05,
             bottom="128-64", hidden="256-64")
_RMC2 = dict(tables=40, rows=2_000_000, dim=64, dtype="f16", dense=256, length=80, lengths="poisson",
             ids="zipf", alpha=1.05, bottom="256-64", hidden="512-128")
_RMC3 = dict(tables=10, rows=1_000_000, dim=32, dtype="f32", dense=2560, length=20, bottom="1024-256-32",
             hidden="512-256")
# The 60-table variant with 4 M instead of 20 M rows a table (31 instead of 154 GB),
# so that several models fit the card side by side.
_LARGE = dict(tables=60, rows=4_000_000, dim=64, dtype="f16", dense=256, length=80, lengths="poisson",
              ids="zipf", alpha=1.2, bottom="256-64", hidden="512-128")
_MTWND = dict(tables=26, rows=1_000_000, dim=64, dtype="f16", dense=64, length=1, ids="zipf", alpha=1.05,
              bottom="", hidden="1024-512-256", interaction="concat", towers=4)


def listed():
    return [
        # Single-item queries on the small model, one call each: nothing but latency and
        # launches (64 calls a pass, so that there are logits enough to compare).
        _case("tiny_b1", batch=1, batches=64, **_TINY),
        # The small model's whole batch.
        _case("tiny_b256", batch=256, **_TINY),
        # Sparse-light model, its batch: fp32 rows, narrow FC stacks.
        _case("rmc1_b1024", batch=1024, **_RMC1),
        # The same from a program that may not allocate (static scratch), at a
        # batch that is no multiple of any tile.
        _case("rmc1_static_b1003", batch=1003, mode="static", **_RMC1),
        # Sparse-heavy model under a tight latency bound: small fused batch.
        _case("rmc2_b256", batch=256, **_RMC2),
        # Sparse-heavy model, its batch, one call after the other: the headline workload.
        _case("rmc2_b4096", batch=4096, **_RMC2),
        # The same through the sparse-dense pipeline, eight batches and a drain:
        # a server that keeps batches in flight.
        _case("rmc2_pipelined_b4096", batch=4096, mode="pipelined", batches=8, **_RMC2),
        # Id streams without reuse, rows loaded past the caches: pooling against
        # HBM; a batch one short of the tile grid.
        _case("rmc2_uniform_b4095", batch=4095, stream_rows=True, **{**_RMC2, "ids": "uniform", "alpha": 0.0}),
        # 60 tables at the largest batch of the batch-size sweep: throughput serving.
        _case("large_b16384", batch=16384, **_LARGE),
        # Dense-heavy model: the 2560-wide Bottom-FC beside short bags.
        _case("rmc3_b4096", batch=4096, **_RMC3),
        # Multi-task model: single lookups, concatenation, four wide towers.
        _case("mtwnd_b4096", batch=4096, **_MTWND),
        # The same at a small odd batch: towers whose weights outweigh their activations.
        _case("mtwnd_b300", batch=300, **_MTWND),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same five model kinds: batch over the whole range, tables,
    rows, lengths and widths around the kind's own."""
    kind = rng.choice(["tiny", "rmc1", "rmc2", "rmc3", "mtwnd"])
    base = dict({"tiny": _TINY, "rmc1": _RMC1, "rmc2": _RMC2, "rmc3": _RMC3, "mtwnd": _MTWND}[kind])
    base["batch"] = _log_int(rng, 1, 6000)
    base["batches"] = max(1, 64 // base["batch"])  # small batches come as a run of calls
    base["rows"] = _log_int(rng, 50_000, 2_000_000)
    base["dtype"] = rng.choice(["f16", "f32"])
    base["ids"], base["alpha"] = rng.choice([("uniform", 0.0), ("zipf", 1.05), ("zipf", 1.2)])
    base["stream_rows"] = base["ids"] == "uniform" and rng.random() < 0.5
    if kind == "mtwnd":
        base["tables"] = rng.randint(4, 28)
        base["dim"] = rng.choice([32, 64])
        base["bottom"] = rng.choice(["", "", "40", "64"])
        base["dense"] = rng.choice([24, 64, 100])
        base["towers"] = rng.randint(1, 4)
        base["hidden"] = rng.choice(["1024-512-256", "512-256", "96-72", "600-200"])
    else:
        base["tables"] = rng.randint(4, 44) if kind == "rmc2" else rng.randint(4, 14)
        base["dim"] = rng.choice([32, 64])
        base["length"] = rng.randint(20, 80) if kind == "rmc2" else rng.randint(8, 80)
        base["lengths"] = rng.choice(["fixed", "poisson"])
        dim = base["dim"]
        if kind == "rmc3":
            base["dense"] = rng.choice([1000, 1536, 2560])
            base["bottom"] = f"1024-256-{dim}"
            base["hidden"] = rng.choice(["512-256", "300-100"])
        elif kind == "tiny":
            base["dense"] = rng.choice([13, 24, 50])
            base["bottom"] = f"256-128-{dim}"
            base["hidden"] = rng.choice(["64", "100-50"])
        else:
            base["dense"] = rng.choice([100, 256, 500])
            base["bottom"] = rng.choice([f"256-{dim}", f"128-{dim}"])
            base["hidden"] = rng.choice(["512-128", "256-64", "200-72"])
    small = base["batch"] * base["tables"] * base["dim"] <= 1_500_000
    base["mode"] = rng.choice(["forward", "forward", "static"]) if small else "forward"
    return _case("", **base)


# ---------------------------------------------------------------------- inputs
def _widths(text):
    return [int(x) for x in text.split("-")] if text else []


def _shapes(case):
    """(bottom widths, top widths) with their inputs, as RecModel takes them."""
    bottom = [case["dense"]] + _widths(case["bottom"])
    t = case["tables"]
    z = bottom[-1] + t * case["dim"] if case["interaction"] == "concat" else case["dim"] + t * (t + 1) // 2
    return bottom, [z] + _widths(case["hidden"]) + [1]


@functools.lru_cache(maxsize=8)
def _zipf_cdf(rows, alpha):
    """CDF of the bounded Zipf law on ranks 1..rows (on the host, so that it is the same everywhere)."""
    c = np.cumsum(np.arange(1, rows + 1, dtype=np.float64) ** -alpha)
    return c / c[-1]


def _scatter(rows, table):
    """rank -> (a * rank + c) mod rows, a bijection without spatial locality."""
    a = (rows * 0.6180339887 + 7919 * (table + 1)) // 1
    a = int(a) % rows or 1
    while math.gcd(a, rows) != 1:
        a += 1
    return a, (104729 * (table + 1)) % rows


def _gen(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1_000_003 + what * 7_919 + 2203) % (1 << 62))
    return g


def _draw_batch(case, seed, k, cdf):
    T, B, rows, dev = case["tables"], case["batch"], case["rows"], "cuda"
    g = _gen(seed, 1000 + k)
    dense = torch.randn((B, case["dense"]), generator=g, device=dev)
    n = T * B
    if case["lengths"] == "fixed":
        lengths = torch.full((n,), case["length"], dtype=torch.int32, device=dev)
    else:
        lam = torch.full((n,), float(case["length"]), device=dev)
        lengths = torch.poisson(lam, generator=g).clamp_(1, 200).to(torch.int32)
    per_table = lengths.view(T, B).sum(dim=1, dtype=torch.int64).tolist()
    parts = []
    for t in range(T):
        if case["ids"] == "uniform":
            parts.append(torch.randint(0, rows, (per_table[t],), generator=g, device=dev, dtype=torch.int32))
        else:
            u = torch.rand(per_table[t], generator=g, device=dev, dtype=torch.float64)
            rank = torch.searchsorted(cdf, u, right=True).clamp_(max=rows - 1)
            a, c = _scatter(rows, t)
            parts.append(((rank * a + c) % rows).to(torch.int32))
    return dense, torch.cat(parts), lengths


def _inputs(case, seed):
    """Tables, per-layer weights and batches, all on the device."""
    tdt = torch.float16 if case["dtype"] == "f16" else torch.float32
    g = _gen(seed, 1)
    tables = [torch.empty((case["rows"], case["dim"]), dtype=tdt, device="cuda").uniform_(-0.05, 0.05, generator=g)
              for _ in range(case["tables"])]
    bottom, top = _shapes(case)
    g = _gen(seed, 2)

    def stack(widths):
        out = []
        for fan_in, fan_out in zip(widths[:-1], widths[1:]):
            W = torch.randn((fan_out, fan_in), generator=g, device="cuda") * fan_in ** -0.5
            b = torch.randn((fan_out,), generator=g, device="cuda") * fan_in ** -0.5
            out.append((W, b))
        return out

    stacks = [stack(bottom)] + [stack(top) for _ in range(case["towers"])]
    cdf = None
    if case["ids"] == "zipf":
        cdf = torch.from_numpy(_zipf_cdf(case["rows"], case["alpha"])).cuda()
    return tables, stacks, [_draw_batch(case, seed, k, cdf) for k in range(case["batches"])]


@functools.lru_cache(maxsize=1)
def _serving_streams():
    """A server creates its streams once and hands them to every pipelined model."""
    return torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()


# ------------------------------------------------------------------- the calls
def prepare(case, seed):
    tables, stacks, batches = _inputs(case, seed)
    bottom, top = _shapes(case)
    max_nnz = max(b[1].numel() for b in batches)
    extra = {}
    if case["mode"] == "pipelined":
        d, p0, p1 = _serving_streams()
        extra = dict(pipeline=True, dense_stream=d, pool_streams=(p0, p1))
    m = binding.RecModel(case["tables"], case["dim"], [case["rows"]] * case["tables"], case["dtype"],
                         case["dense"], bottom, top, case["batch"], max_nnz,
                         interaction=case["interaction"], towers=case["towers"], **extra)
    for t, tab in enumerate(tables):
        m.load_table(t, tab)
    for k, stack in enumerate(stacks):
        for i, (W, b) in enumerate(stack):
            m.load_mlp(binding.REC_BOTTOM if k == 0 else binding.REC_TOP + k - 1, i, W, b)
    if case["stream_rows"]:
        m.set_option(binding.REC_OPT_STREAM_ROWS, 1)
    shape = (case["batch"],) if case["towers"] == 1 else (case["batch"], case["towers"])
    logits = torch.empty((case["batches"],) + shape, device="cuda")
    return dict(model=m, batches=batches, logits=logits, outs=list(logits), mode=case["mode"],
                fault=torch.zeros(2, dtype=torch.int64, device="cuda"))


def run(state):
    m = state["model"]
    for (dense, ids, lengths), out in zip(state["batches"], state["outs"]):
        if state["mode"] == "static":
            m.forward_static(dense, ids, lengths, out, state["fault"])
        else:
            m.forward(dense, ids, lengths, out)
    if state["mode"] == "pipelined":
        m.drain()
    return state["logits"]


# ----------------------------------------------------------- what they are worth
def work(case):
    """Distinct rows touched, ids, lengths, dense features and weights (bf16) read
    once, logits written once; multiply-adds of pooling, interaction and FC layers."""
    T, B, D = case["tables"], case["batch"], case["dim"]
    ids_per_table = B * case["length"]
    if case["ids"] == "uniform":
        distinct = case["rows"] * -math.expm1(ids_per_table * math.log1p(-1.0 / case["rows"]))
    else:
        p = np.diff(_zipf_cdf(case["rows"], case["alpha"]), prepend=0.0)
        distinct = float(-np.expm1(ids_per_table * np.log1p(-p)).sum())
    bottom, top = _shapes(case)
    macs = sum(a * b for a, b in zip(bottom[:-1], bottom[1:]))
    macs += case["towers"] * sum(a * b for a, b in zip(top[:-1], top[1:]))
    elt = 2 if case["dtype"] == "f16" else 4
    per_batch = T * distinct * D * elt + 4 * T * ids_per_table + 4 * T * B + 4 * B * case["dense"] + 4 * B * case["towers"]
    inter = T * (T + 1) // 2 * D if case["interaction"] == "dot" else 0
    flops = B * (2 * (macs + inter) + T * case["length"] * D)
    return {"bytes": case["batches"] * per_batch + 2 * macs, "flops": case["batches"] * flops}


def tolerance(case):
    # Every matrix layer narrows its operands to bf16, and so does the interaction its
    # output: sums taken in another order land on the other side of a rounding
    # boundary here and there.  The same narrowing with sums in 64 bits differs
    # from this library by up to 9.3e-4 (2-norm) and 1.25e-2 (largest) over the
    # listed and 24 drawn cases; four times that.
    return {"rel": 4e-3, "max": 5e-2}


def exact(case, seed):
    """The same forward in 64 bits: plain torch, no narrowing anywhere."""
    tables, stacks, batches = _inputs(case, seed)
    T, B, D = case["tables"], case["batch"], case["dim"]

    def layers(x, stack, last_linear):
        for i, (W, b) in enumerate(stack):
            x = x @ W.double().t().contiguous() + b.double()
            if not (last_linear and i == len(stack) - 1):
                x = x.clamp_(min=0.0)
        return x

    outs = []
    for dense, ids, lengths in batches:
        x0 = layers(dense.double(), stacks[0], False)
        lens = lengths.view(T, B).to(torch.int64)
        vecs, at = [], 0
        for t in range(T):
            n = int(lens[t].sum())
            bag = torch.repeat_interleave(torch.arange(B, device="cuda"), lens[t])
            sums = torch.zeros((B, D), dtype=torch.float64, device="cuda")
            sums.index_add_(0, bag, tables[t][ids[at:at + n].long()].double())
            vecs.append(sums)
            at += n
        if case["interaction"] == "concat":
            z = torch.cat([x0] + vecs, dim=1)
        else:
            X = torch.stack([x0] + vecs, dim=1)
            i, j = torch.tril_indices(T + 1, T + 1, offset=-1, device="cuda")
            parts = []
            for lo in range(0, B, 2048):
                x = X[lo:lo + 2048]
                parts.append(torch.bmm(x, x.transpose(1, 2).contiguous())[:, i, j])
            z = torch.cat([x0, torch.cat(parts)], dim=1)
        logits = [layers(z, s, True)[:, 0] for s in stacks[1:]]
        outs.append(logits[0] if case["towers"] == 1 else torch.stack(logits, dim=1))
    return torch.stack(outs)
