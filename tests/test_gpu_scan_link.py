"""The scan in one launch: its blocks hand their tiles' sums to the later ones through
words that each launch leaves as it found them.  Offsets exact for batches of one
to 300 tiles, call after call on one model with other batch sizes in between, with
Bottom-FC riding along, alone, and in a graph replayed over changing lengths."""
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


def layer(g, n, k):
    return [((g.standard_normal((n, k)) * k ** -0.5).astype(np.float32), np.zeros(n, np.float32))]


def model(binding, g, interaction, T, D, R, B, F, nnz):
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float32) for _ in range(T)]
    dot = interaction == "dot"
    width = D + T * (T + 1) // 2 if dot else F + T * D
    return H.make_model(binding, tabs, layer(g, D, F) if dot else [], layer(g, 1, width), B, nnz, F,
                        interaction=interaction)


@pytest.mark.parametrize("interaction", ["dot", "concat"])
def test_offsets_call_after_call(binding, interaction):
    g = np.random.default_rng(960)
    T, D, R, F, most = 6, 4, 50, 5, 102_400
    m = model(binding, g, interaction, T, D, R, most, F, T * most * 3)
    for B in (102_400, 342, 683, 102_399, 1, 3000, 102_400, 50_000):   # 300, 2 (just past), 3, ..., 147 tiles
        print("linked scan", interaction, B, flush=True)
        lens = g.integers(0, 3, T * B).astype(np.int32)
        idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
        dense = g.standard_normal((B, F)).astype(np.float32)
        H.run(m, synth.Batch(dense, idx, lens))
        assert m.check() == (binding.REC_OK, -1)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), orc.offsets(lens)[0])
    neg = lens.copy()
    neg[[-5000, -3]] = (-7, -1)
    keep = int(np.maximum(neg, 0).sum())
    H.run(m, synth.Batch(dense, idx[:keep], neg))
    assert m.check() == (binding.REC_ERR_LENGTHS, neg.size - 5000)
    assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), orc.offsets(neg)[0])
    m.close()


def test_offsets_of_graph_replays(binding):
    print("linked scan, graph", flush=True)
    g = np.random.default_rng(961)
    T, D, R, F, B, nnz = 9, 4, 50, 5, 20_000, 180_000      # 88 tiles
    m = model(binding, g, "concat", T, D, R, B, F, nnz)
    dense = torch.from_numpy(g.standard_normal((B, F)).astype(np.float32)).cuda()
    idx = torch.from_numpy(g.integers(0, R, nnz).astype(np.int32)).cuda()

    def lengths():  # nnz ids spread over the bags in another way each time
        return np.bincount(g.integers(0, T * B, nnz), minlength=T * B).astype(np.int32)
    lens = torch.from_numpy(lengths()).cuda()
    out = torch.empty(B, dtype=torch.float32, device="cuda")
    m.forward(dense, idx, lens, out)
    cap = binding.CapturedForward(m, [(dense, idx, lens)], [out])
    for _ in range(4):
        now = lengths()
        lens.copy_(torch.from_numpy(now))
        cap.replay()
        torch.cuda.synchronize()
        assert m.check() == (binding.REC_OK, -1)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), orc.offsets(now)[0])
        got = out.clone()
        m.forward(dense, idx, lens, out)             # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(got, out)
    m.close()
