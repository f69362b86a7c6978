"""FC stacks run as chains (several layers in one kernel, activations on chip)
against the CPU oracle, and against the same stacks run layer by layer.

Both device paths narrow the same operands to bf16 and differ only in the
order of the fp32 sums, so each is held to the oracle's bars (2e-2 relative on
the batch against the exact forward, 5e-3 per sample against the bf16 mirror)
and the two are held to each other more tightly (1e-3).
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import rec_oracle as orc
from paper_2203_07424_amd import synth

import gpu_helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2203_07424_amd import binding as b
    return b


def say(*a):
    print(*a, flush=True)


def stack(g, ws):
    return [((g.standard_normal((ws[i + 1], ws[i])) * ws[i] ** -0.5).astype(np.float32),
             (g.standard_normal(ws[i + 1]) * ws[i] ** -0.5).astype(np.float32))
            for i in range(len(ws) - 1)]


def check(got, exact, mirror, other=None):
    """The oracle's bars, with the per-sample mirror bar read for deep stacks: a
    sum that falls next to a bf16 rounding boundary may round the other way on
    the device (fp32 sums) than in the mirror (fp64 sums), and a narrow layer
    further down can carry that one-ulp difference into a logit.  So 98 % of the
    samples meet 5e-3 and every sample 2e-2.  The two device paths narrow the
    same operands and differ in the order of fp32 sums only."""
    got = got.astype(np.float64)
    if got.ndim == 2:
        for k in range(got.shape[1]):
            check(got[:, k], exact[:, k], mirror[:, k], None if other is None else other[:, k])
        return
    if got.size >= 8:
        H.check_logits(got, exact)
    scale = np.maximum(np.abs(mirror), float(np.sqrt((mirror ** 2).mean())))
    err = np.abs(got - mirror) / scale
    assert err.max() <= 2e-2 and np.quantile(err, 0.98) <= 5e-3, (err.max(), np.quantile(err, 0.98))
    if other is not None:
        gap = np.abs(got - other.astype(np.float64)) / scale
        assert gap.max() <= 2e-2 and np.quantile(gap, 0.98) <= 1e-3, (gap.max(), np.quantile(gap, 0.98))


def both_ways(binding, m, batch):
    m.set_option(binding.REC_OPT_FUSE_MLP, 2)
    fused = H.run(m, batch)
    fused_x0 = m.debug_bottom_out().cpu().numpy() if m.n_bottom else None
    m.set_option(binding.REC_OPT_FUSE_MLP, 0)
    plain = H.run(m, batch)
    plain_x0 = m.debug_bottom_out().cpu().numpy() if m.n_bottom else None
    m.set_option(binding.REC_OPT_FUSE_MLP, 2)
    again = H.run(m, batch)
    m.set_option(binding.REC_OPT_FUSE_MLP, 1)
    auto = H.run(m, batch)                       # the library's own choice per run: one of the two
    assert np.array_equal(auto, fused) or np.array_equal(auto, plain) or \
        np.abs(auto - fused).max() <= 2e-2 * max(np.abs(fused).max(), 1e-6)
    assert np.array_equal(fused, again)          # fixed order of sums: reproducible
    assert m.check() == (binding.REC_OK, -1)
    return fused, plain, fused_x0, plain_x0


DOT_CASES = [
    # T, R, D, dtype, B, F, bottom hidden, top hidden
    (3, 300, 32, np.float32, 70, 13, (40,), (24,)),                  # ragged widths, unaligned dense rows
    (4, 200, 64, np.float16, 1, 8, (64, 64), (64,)),                 # one sample
    (8, 300, 64, np.float16, 33, 256, (256,), (512, 128)),           # one row past a block of 32
    (5, 200, 32, np.float32, 200, 100, (1000, 1024, 70), (1024, 1000, 33, 64)),   # the widest layers a chain takes
    (3, 200, 16, np.float16, 95, 20, (30, 40, 50, 60, 70, 80, 90), (100, 90, 80, 70, 60, 50, 40, 30)),  # longer than one chain
    (3, 200, 32, np.float32, 130, 1500, (600, 1100, 200), (300, 1200, 1100, 64)),  # wide layers between chains
    (2, 100, 32, np.float16, 64, 4, (), (300,)),                     # no Bottom-FC
]


@pytest.mark.parametrize("T,R,D,dtype,B,F,hb,ht", DOT_CASES)
def test_chained_stacks_against_oracle_and_per_layer_path(binding, T, R, D, dtype, B, F, hb, ht):
    say("chain case", T, R, D, dtype.__name__, B, F, hb, ht)
    g = np.random.default_rng(900 + T + B)
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    lens = g.integers(0, 30, T * B).astype(np.int32)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    if hb:
        bottom = stack(g, (F,) + tuple(hb) + (D,))
    else:
        F, bottom = D, []
    top = stack(g, (D + T * (T + 1) // 2,) + tuple(ht) + (1,))
    dense = g.standard_normal((B, F)).astype(np.float32)
    m = H.make_model(binding, tabs, bottom, top, B + 3, max(idx.size, 1), F)
    m.n_bottom = len(bottom)
    batch = synth.Batch(dense, idx, lens)
    fused, plain, fx0, px0 = both_ways(binding, m, batch)
    exact = orc.forward(dense, tabs, idx, lens, bottom, top)
    mirror = orc.forward(dense, tabs, idx, lens, bottom, top, orc.BF16_MIRROR)
    check(fused, exact["logits"], mirror["logits"], plain)
    check(plain, exact["logits"], mirror["logits"])
    if bottom:
        for x0 in (fx0, px0):
            x0 = x0[:B, :D].astype(np.float64)
            ref = mirror["bottom_out"]
            assert np.abs(x0 - ref).max() <= 5e-3 * max(np.abs(ref).max(), 1e-6)
    m.close()


TOWER_CASES = [
    # T, R, D, dtype, B, F, bottom hidden, tower hidden, towers
    (5, 300, 32, np.float32, 70, 24, (40,), (96, 72), 3),
    (26, 300, 64, np.float16, 130, 64, (), (1024, 512, 256), 4),     # the MT-WnD stack: wide first layer, chain behind it
    (3, 100, 32, np.float16, 90, 8, (), (40, 300), 8),
    (2, 100, 8, np.float32, 257, 5, (), (), 5),                      # towers of one (one-output) layer
    (4, 100, 64, np.float16, 100, 16, (), (1100, 64, 1100, 64), 2),  # chains between wide layers, per tower
]


@pytest.mark.parametrize("T,R,D,dtype,B,F,hb,ht,nt", TOWER_CASES)
def test_chained_towers_against_oracle_and_per_layer_path(binding, T, R, D, dtype, B, F, hb, ht, nt):
    say("chain towers", T, R, D, dtype.__name__, B, F, hb, ht, nt)
    g = np.random.default_rng(950 + T + B)
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    lens = np.ones(T * B, np.int32)
    idx = g.integers(0, R, T * B).astype(np.int32)
    bottom = stack(g, (F,) + tuple(hb)) if hb else []
    w0 = hb[-1] if hb else F
    towers = [stack(g, (w0 + T * D,) + tuple(ht) + (1,)) for _ in range(nt)]
    dense = g.standard_normal((B, F)).astype(np.float32)
    m = H.make_model(binding, tabs, bottom, towers, B, idx.size, F, interaction="concat")
    m.n_bottom = len(bottom)
    fused, plain, _, _ = both_ways(binding, m, synth.Batch(dense, idx, lens))
    exact = orc.forward_towers(dense, tabs, idx, lens, bottom, towers, orc.EXACT)
    mirror = orc.forward_towers(dense, tabs, idx, lens, bottom, towers, orc.BF16_MIRROR)
    check(fused, exact["logits"], mirror["logits"], plain)
    check(plain, exact["logits"], mirror["logits"])
    m.close()


def test_chain_in_a_graph_and_beside_pooling(binding):
    # The chain kernels under HIP graph replay and on the side stream.
    say("chain graph/overlap")
    g = np.random.default_rng(77)
    T, R, D, B, F = 6, 400, 32, 150, 48
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    lens = g.integers(0, 50, T * B).astype(np.int32)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    bottom = stack(g, (F, 128, 64, D))
    top = stack(g, (D + T * (T + 1) // 2, 256, 96, 1))
    dense = g.standard_normal((B, F)).astype(np.float32)
    m = H.make_model(binding, tabs, bottom, top, B, idx.size, F)
    m.set_option(binding.REC_OPT_FUSE_MLP, 2)
    batch = synth.Batch(dense, idx, lens)
    eager = H.run(m, batch)
    m.set_option(binding.REC_OPT_OVERLAP_DENSE, 1)
    assert np.array_equal(H.run(m, batch), eager)
    m.set_option(binding.REC_OPT_OVERLAP_DENSE, 0)
    d, i, l = (torch.from_numpy(x).cuda() for x in (dense, idx, lens))
    out = torch.empty(B, dtype=torch.float32, device="cuda")
    cap = binding.CapturedForward(m, [(d, i, l)], [out])
    for _ in range(3):
        out.zero_()
        cap.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), eager)
        assert np.array_equal(H.run(m, batch), eager)      # eager work between the replays
    mirror = orc.forward(dense, tabs, idx, lens, bottom, top, orc.BF16_MIRROR)
    exact = orc.forward(dense, tabs, idx, lens, bottom, top)
    H.check_logits(eager, exact["logits"], mirror["logits"])
    m.close()


@pytest.mark.parametrize("name", ["rmc2", "rmc1", "mtwnd"])
def test_full_size_workload_with_every_possible_chain(binding, name):
    """The named workload at full size with chains forced wherever the layer
    shapes allow (by itself the library chains only the narrow stacks); the
    oracle recomputes a spread of samples."""
    w = synth.WORKLOADS[name]
    say("full-size workload, chains forced", name)
    m, bottom, top = H.make_workload_model(binding, w)
    m.set_option(binding.REC_OPT_FUSE_MLP, 2)
    batch = synth.draw_batch(w, 0)
    forced = H.run(m, batch)
    assert m.check() == (binding.REC_OK, -1)
    m.set_option(binding.REC_OPT_FUSE_MLP, 0)
    plain = H.run(m, batch)
    g = np.random.default_rng(6)
    pick = np.unique(np.concatenate([[0, 1, 31, 32, w.batch - 33, w.batch - 1], g.integers(0, w.batch, 40)]))
    exact = H.oracle_on_slice(w, batch, pick, bottom, top)
    mirror = H.oracle_on_slice(w, batch, pick, bottom, top, orc.BF16_MIRROR)
    check(forced[pick], exact["logits"], mirror["logits"], plain[pick])
    assert np.isfinite(forced).all()
    m.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name,B", [("tiny", 256), ("tiny", 1), ("tiny", 77), ("rmc1", 1024), ("rmc2", 4096)])
def test_bottom_fc_riding_on_the_scan_equals_its_own_launch(binding, name, B):
    """An in-order forward runs a chainable Bottom-FC inside the scan's second
    launch.  With REC_OPT_OVERLAP_DENSE the same stack is a launch of its own (on
    the side stream): same kernel body, same sums, so the bits must agree - for
    the Bottom-FC output and for the logits - and the offsets must still be right."""
    w = synth.WORKLOADS[name].with_batch(B)
    say("Bottom-FC on the scan", name, B)
    ride, _, _ = H.make_workload_model(binding, w)
    own, _, _ = H.make_workload_model(binding, w, share_tables=ride)
    own.set_option(binding.REC_OPT_OVERLAP_DENSE, 1)
    for seed in (3, 4):
        b = synth.draw_batch(w, seed)
        d = [torch.from_numpy(a).cuda() for a in (b.dense, b.indices, b.lengths)]
        got, want = ride.forward(*d), own.forward(*d)
        torch.cuda.synchronize()
        assert ride.check() == (binding.REC_OK, -1) and own.check() == (binding.REC_OK, -1)
        assert torch.equal(ride.debug_bottom_out(), own.debug_bottom_out())
        assert torch.equal(got, want)
        assert np.array_equal(np.diff(ride.debug_offsets().cpu().numpy().astype(np.int64)), b.lengths)
    ride.close()
    own.close()
    torch.cuda.empty_cache()


def test_stage_timing_says_where_bottom_fc_ran(binding):
    """In order, a chainable Bottom-FC has no launch of its own: both of its stages
    read 0 and the scan's stage holds it.  Layer by layer (REC_OPT_FUSE_MLP = 0)
    every stage has an interval of its own."""
    w = synth.WORKLOADS["tiny"]
    say("stage timing, Bottom-FC on the scan")
    m, _, _ = H.make_workload_model(binding, w)
    b = synth.draw_batch(w, 9)
    d = [torch.from_numpy(a).cuda() for a in (b.dense, b.indices, b.lengths)]
    for fuse, riding in ((1, True), (0, False)):
        m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
        m.set_profiling(2, 1)
        for _ in range(2):
            m.forward(*d)
        torch.cuda.synchronize()
        for slot in range(2):
            ms = m.stage_ms(slot)
            for k, v in ms.items():
                if riding and k in ("bottom_first", "bottom_rest"):
                    assert v == 0.0, ms
                else:
                    assert v > 0.0, ms
        m.set_profiling(0)
    m.close()


@pytest.mark.parametrize("name,B,fuse,pipelined,shared", [
    ("tiny", 256, 1, False, {"scan", "bottom_first", "bottom_rest", "interact", "top_rest"}),   # two launches
    ("tiny", 2000, 1, False, {"bottom_first", "bottom_rest", "interact", "top_rest"}),          # too many bags for the first
    ("tiny", 256, 0, False, {"top_rest"}),                                                      # one hidden layer, dot folded in
    ("tiny", 256, 2, True, {"bottom_rest", "interact", "top_rest"}),
    ("mtwnd-tiny", 200, 1, False, {"bottom_rest", "top_rest"}),
    ("mtwnd", 64, 1, False, {"scan", "bottom_first", "bottom_rest", "interact"}),               # no Bottom-FC
    ("rmc2", 256, 1, False, {"bottom_first", "bottom_rest"}),
    ("rmc2", 4096, 1, False, {"bottom_first", "bottom_rest", "interact", "top_rest"}),
])
def test_stages_that_share_a_launch_are_named(binding, name, B, fuse, pipelined, shared):
    w = synth.WORKLOADS[name].with_batch(B)
    if w.rows > 100_000:
        w = dataclasses.replace(w, rows=100_000)
    say("stages sharing a launch", name, B, fuse, pipelined)
    m, _, _ = H.make_workload_model(binding, w, pipeline=pipelined)
    m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
    b = synth.draw_batch(w, 9)
    d = [torch.from_numpy(a).cuda() for a in (b.dense, b.indices, b.lengths)]
    assert binding.rec_stage_shared(m.handle)[0] == binding.REC_ERR_STATE
    m.set_profiling(2, 1)
    m.forward(*d)
    m.drain()
    torch.cuda.synchronize()
    assert m.stage_shared(0) == shared
    assert binding.rec_stage_shared(m.handle, 1)[0] == binding.REC_ERR_STATE
    m.set_profiling(0)
    m.close()


@pytest.mark.parametrize("hidden,rounds,chained", [
    ((256, 256), 1, False), ((256, 128), 1, False), ((256,) * 5, 1, True), ((512, 256), 1, True), ((64, 64), 1, True),
    ((512, 256), 2, False), ((512, 512), 2, True), ((1024, 256), 2, True), ((256,) * 5, 2, True)])
def test_heavy_runs_are_chained_where_that_saves_launches(binding, hidden, rounds, chained):
    """1024 inputs, four towers, blocks of 64 samples for every compute unit once or
    twice: runs with a wide layer are chained whatever their weights (twice: if that
    saves two launches or more than 512 columns of activations), narrow ones (blocks
    of 32) up to 256 KiB a launch saved."""
    say("heavy runs", hidden, rounds)
    g = np.random.default_rng(990)
    T, R, D, F, nt = 15, 40, 64, 64, 4
    B = 16 * rounds * torch.cuda.get_device_properties(0).multi_processor_count
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    towers = [stack(g, (F + T * D,) + hidden + (1,)) for _ in range(nt)]
    m = H.make_model(binding, tabs, [], towers, B, T * B, F, interaction="concat")
    idx = g.integers(0, R, T * B).astype(np.int32)
    d = [torch.from_numpy(a).cuda() for a in (g.standard_normal((B, F)).astype(np.float32), idx, np.ones(T * B, np.int32))]
    m.set_profiling(1, 1)
    m.forward(*d)
    torch.cuda.synchronize()
    assert m.check() == (binding.REC_OK, -1)
    assert ("top_rest" in m.stage_shared(0)) == chained
    m.set_profiling(0)
    m.close()


@pytest.mark.parametrize("B", [300, 1000, 1024, 1100])
def test_short_scan_in_one_launch_with_faults(binding, B):
    """Up to 8 scan tiles with a Bottom-FC riding along: the scan is one launch
    whose blocks add up the earlier lengths themselves.  Offsets bit-exact, a
    negative length in a later tile and a wrong total reported as ever."""
    w = synth.WORKLOADS["tiny"].with_batch(B)          # 8 tables: 2, 4, 4 and 5 tiles
    say("one-launch scan", B)
    m, _, _ = H.make_workload_model(binding, w)
    b = synth.draw_batch(w, 21)
    off, rc, _ = orc.offsets(b.lengths)
    assert rc == 0
    H.run(m, b)
    assert m.check() == (binding.REC_OK, -1)
    assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
    # a negative length in the last tile: counted as zero, its position reported
    neg = b.lengths.copy()
    at = neg.size - 7
    cut = int(neg[at])
    neg[at] = -cut - 1
    start = int(b.lengths[:at].sum())
    idx = np.concatenate([b.indices[:start], b.indices[start + cut:]])
    H.run(m, synth.Batch(b.dense, idx, neg))
    off2, rc2, bad = orc.offsets(neg)
    assert rc2 == -1 and bad == at
    assert m.check() == (binding.REC_ERR_LENGTHS, at)
    assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off2)
    # total != nnz: reported, offsets clamped
    logits = H.run(m, synth.Batch(b.dense, b.indices[:-5], b.lengths))
    assert m.check() == (binding.REC_ERR_LENGTHS, -1)
    assert np.isfinite(logits).all()
    assert m.debug_offsets().cpu().numpy().max() == b.indices.size - 5
    m.close()
