"""The first Bottom-FC layer beside scan and pooling (small batches) or beside the
scan, in each block tile it comes in, at their edges; in a concatenation model it
writes its columns of the Predict-FC input rows as well.

A forward whose stages are timed gives the layer and the scan launches of their own,
with the same order of sums: every buffer is the same bits.  Offsets, sums and logits
are held to the oracle as everywhere."""
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


def stack(g, ws):
    return [((g.standard_normal((ws[i + 1], ws[i])) * ws[i] ** -0.5).astype(np.float32),
             (g.standard_normal(ws[i + 1]) * ws[i] ** -0.5).astype(np.float32))
            for i in range(len(ws) - 1)]


def buffers(m, batch, concat):
    logits = H.run(m, batch)
    return [torch.from_numpy(logits), m.debug_offsets().clone(), m.debug_bottom_out().clone(), m.debug_interact().clone()] + \
        ([] if concat else [m.debug_pooled().clone()])


def spoil(binding, m, byte):
    """What the forward is to overwrite: Bottom-FC's output and the Predict-FC input."""
    for what, size in ((binding.REC_DBG_BOTTOM_OUT, 4), (binding.REC_DBG_INTERACT, 2)):
        _, _, ld = binding.rec_debug_get(m.handle, what)
        m._view(what, size * m.last_batch * ld)[0].fill_(byte)


def compare(binding, m, batch, concat=False):
    """One forward in joint launches against the same in launches of their own."""
    H.run(m, batch)
    spoil(binding, m, 0x41)
    joint = buffers(m, batch, concat)
    spoil(binding, m, 0x42)
    m.set_profiling(1, 1)
    apart = buffers(m, batch, concat)
    m.set_profiling(0)
    assert m.check() == (binding.REC_OK, -1)
    assert all(torch.equal(a, b) for a, b in zip(joint, apart))
    off, _, _ = orc.offsets(batch.lengths)
    assert np.array_equal(joint[1].cpu().numpy().astype(np.int64), off)
    return joint


# where: the launch that has the layer, "joined": that of the scan with pooling in it too; tile: its rows, columns and the waves that share its
# k on 256 compute units (128 x 128: csrc/gemm_big.hip).
POOLED = [
    (1, 32, np.float32, 1, 2560, (1024, 256), 20, "pooling", (16, 16, 8)),
    (10, 32, np.float16, 17, 1000, (1024, 256), 20, "pooling", (16, 16, 8)),
    (10, 64, np.float32, 113, 1000, (1024, 256), 8, "pooling", (16, 32, 8)),
    (11, 32, np.float32, 223, 1000, (1024, 256), 10, "pooling", (32, 32, 8)),
    (9, 32, np.float16, 195, 2560, (1024, 256), 9, "pooling", (32, 32, 8)),
    (8, 64, np.float16, 895, 500, (256,), 12, "pooling", (32, 32, 4)),          # the largest batches
    (10, 32, np.float32, 301, 2560, (1024, 256), 9, "pooling", (32, 64, 8)),
    (7, 32, np.float32, 1001, 1536, (1024, 256), 8, "pooling", (32, 64, 4)),
    (2, 64, np.float32, 1024, 1000, (512, 64), 9, "pooling", (32, 64, 4)),
    (9, 64, np.float16, 797, 500, (256,), 12, "scan", (32, 32, 4)),             # one tile of lengths more
    (10, 32, np.float32, 901, 1536, (1024, 256), 8, "scan", (32, 64, 4)),
    (30, 32, np.float16, 601, 1000, (1024, 256), 9, "scan", (48, 64, 8)),       # 9 tiles of lengths: their sums handed on
    (10, 32, np.float32, 751, 2560, (1024, 256), 8, "scan", (48, 64, 8)),
    (4, 32, np.float32, 1601, 1536, (1024, 256), 8, "scan", (64, 64, 4)),       # few bags, but 64 KB of LDS a block
    (4, 32, np.float16, 1793, 1000, (1024, 256), 8, "scan", (64, 64, 4)),
    (10, 64, np.float32, 2047, 600, (1024, 256), 8, "scan", (64, 64, 4)),
    (5, 32, np.float32, 1187, 1000, (1024, 256), 8, "scan", (80, 64, 8)),
    (12, 16, np.float32, 100, 640, (1024, 32), 9, "pooling", (16, 32, 8)),      # rows of 64 bytes
    (12, 8, np.float16, 100, 640, (1024, 32), 9, "scan", (16, 32, 8)),          # 16-byte rows: never with pooling
    (5, 32, np.float32, 3500, 1536, (1024, 256), 8, "joined", (128, 128, 1)),   # 224 tiles, pooling in the launch too
    (4, 32, np.float32, 2049, 1000, (1024, 256), 7, "joined", (128, 128, 1)),   # 136
    (9, 32, np.float32, 4097, 1000, (1024, 256), 6, "joined", (128, 128, 1)),
    (30, 32, np.float32, 2100, 2560, (1024, 256), 6, "scan", (128, 128, 1)),    # 247 bags a compute unit, 31 tiles of lengths: their sums handed on
    (12, 32, np.float16, 2049, 1000, (1024, 256), 2, "scan", (128, 128, 1)),    # a few ids a bag, 13 tiles
    (3, 32, np.float32, 2500, 1536, (1024, 256), 60, "scan", (128, 128, 1)),    # long bags, 4 tiles: all earlier lengths added up
    (3, 64, np.float32, 65, 300, (), 7, "pooling", (16, 16, 8)),                # the layer is the whole stack
    (6, 32, np.float32, 70, 1501, (1024, 256), 7, None, None),                  # rows that are not read in vectors
]


@pytest.mark.parametrize("T,D,dtype,B,F,bottom,mean,where,tile", POOLED)
def test_layer_of_a_pooled_model(binding, T, D, dtype, B, F, bottom, mean, where, tile):
    print("first layer", T, D, np.dtype(dtype).name, B, F, bottom, flush=True)
    g = np.random.default_rng(1500 + T + B)
    R = 300
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    lens = g.integers(1, 2 * mean, T * B).astype(np.int32)
    lens[:3] = (90, 0, 71)[:min(3, lens.size)]
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    mlp, top = stack(g, (F,) + bottom + (D,)), stack(g, (D + T * (T + 1) // 2, 200, 72, 1))
    m = H.make_model(binding, tabs, mlp, top, B, idx.size, F)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus == 256:
        _, mask, _ = binding.rec_probe_plan(m.handle, B, idx.size)
        assert bool(mask & binding.REC_PLAN_LAYER) == (where is not None)
        assert bool(mask & binding.REC_PLAN_FRONT) == (where not in ("scan", "joined"))
        assert binding.rec_probe_plan_joined(m.handle, B, idx.size) == (binding.REC_OK, where == "joined")
        form = binding.rec_probe_fc_form(B, F, (bottom + (D,))[0], 1, binding.REC_FC_ANY_ORDER | binding.REC_FC_F32_ROWS)[1]
        assert tile is None or form[1:] == tile
    dense = g.standard_normal((B, F)).astype(np.float32)
    batch = synth.Batch(dense, idx, lens)
    logits, _, x0, _, pooled = compare(binding, m, batch)
    P, A, _, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
    H.check_pooled(pooled.cpu().numpy(), P, A)
    if B >= 8:
        H.check_logits(logits.numpy(), orc.forward(dense, tabs, idx, lens, mlp, top, orc.EXACT)["logits"])
    m.set_option(binding.REC_OPT_STREAM_ROWS, 1)
    assert torch.equal(compare(binding, m, batch)[4], pooled)
    m.set_option(binding.REC_OPT_STREAM_ROWS, 0)
    out, fault = torch.empty(B, device="cuda"), torch.zeros(2, dtype=torch.int64, device="cuda")
    m.forward_static(*[torch.from_numpy(a).cuda() for a in (dense, idx, lens)], out, fault)
    assert torch.equal(out.cpu(), logits) and fault.tolist() == [binding.REC_OK, -1]
    bad = idx.copy()
    bad[[3, idx.size - 1]] = (-1, R)
    H.run(m, synth.Batch(dense, bad, lens))
    assert m.check() == (binding.REC_ERR_INDEX_RANGE, 3)
    H.run(m, synth.Batch(dense, idx[:-2], lens))
    assert m.check() == (binding.REC_ERR_LENGTHS, -1)
    assert all(torch.equal(a, b) for a, b in zip(compare(binding, m, batch), (logits, m.debug_offsets(), x0)))
    m.close()


@pytest.mark.parametrize("T,D,dtype,B,F,w0", [
    (5, 32, np.float32, 1, 24, 40), (16, 32, np.float16, 38, 100, 42), (26, 64, np.float16, 300, 64, 64),
    (4, 32, np.float32, 3072, 16, 13), (3, 64, np.float16, 17, 128, 250), (1, 32, np.float16, 8200, 8, 64),  # many tiles: apart
    (1, 64, np.float16, 12289, 20, 64), (26, 64, np.float16, 1501, 64, 33), (6, 16, np.float32, 50, 37, 40),
    (5, 128, np.float32, 40, 64, 40), (26, 64, np.float16, 300, 256, 64),  # a unit of k for each of four waves
    (26, 64, np.float16, 300, 257, 64), (26, 64, np.float16, 300, 260, 64), (26, 64, np.float16, 100, 1000, 200),
    (5, 32, np.float32, 2001, 512, 64)])  # more than one
def test_layer_of_a_concatenation_model(binding, T, D, dtype, B, F, w0):
    print("first layer, concat", T, D, np.dtype(dtype).name, B, F, w0, flush=True)
    g = np.random.default_rng(1600 + T + B)
    R = 200
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    mlp, tops = stack(g, (F, w0)), [stack(g, (w0 + T * D, 96, 1)) for _ in range(2)]
    m = H.make_model(binding, tabs, mlp, tops, B, 4 * T * B, F, interaction="concat")
    dense = g.standard_normal((B, F)).astype(np.float32)
    for lens in (np.ones(T * B, np.int32), g.integers(0, 4, T * B).astype(np.int32)):
        lens[0] = max(int(lens[0]), 1)
        idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
        logits, _, x0, z = compare(binding, m, synth.Batch(dense, idx, lens), concat=True)
        assert torch.equal(z[:, :w0], x0[:, :w0].bfloat16()) and not z[:, w0 + T * D:].any()
        assert not x0[:, w0:].any()
        if B >= 8:
            H.check_logits(logits.numpy(), orc.forward_towers(dense, tabs, idx, lens, mlp, tops, orc.EXACT)["logits"])
    m.close()
