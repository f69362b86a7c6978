"""Scan and pooling in the launch of a wide first layer: row sizes, bags that fill no block and fours that cross
tables, ids of four bags that just fit and do not, empty bags, faults.  Against a timed forward, which gives the three
launches of their own with the same order of sums (every buffer the same bits), and the oracle."""
import numpy as np
import pytest
import torch

from oracle import rec_oracle as orc
from paper_2203_07424_amd import synth

import gpu_helpers as H
from test_gpu_first_layer import compare, stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2203_07424_amd import binding as b
    return b


@pytest.mark.parametrize("T,D,dtype,B,F,stream", [
    (4, 16, np.float32, 2049, 1000, False), (5, 32, np.float16, 2600, 648, True),     # 64-byte rows
    (3, 32, np.float32, 3071, 1000, True), (23, 64, np.float16, 2111, 1536, False),   # 128: the most bags of a block by its LDS
    (9, 64, np.float32, 4097, 2560, False), (3, 128, np.float16, 2303, 1000, True),   # 256
    (29, 32, np.float32, 2118, 2560, False)])                                         # 240 bags a compute unit
def test_pooling_beside_a_wide_layer(binding, T, D, dtype, B, F, stream):
    print("beside wide", T, D, np.dtype(dtype).name, B, F, stream, flush=True)
    g = np.random.default_rng(70 + T + B)
    R, n = 400, T * B
    tabs = [(g.uniform(-1, 1, (R, D)) * 2.0 ** g.integers(-8, 1, (R, D))).astype(dtype) for _ in range(T)]
    lens = g.integers(0, 13, n).astype(np.int32)
    # fours of 256 and 257 ids, one bag of all of them, lengths around the rows of a load and of three
    lens[:24] = (64, 64, 64, 64, 64, 65, 64, 64, 0, 256, 0, 0, 300, 0, 0, 1, 47, 48, 49, 0, 11, 12, 13, 25)
    lens[B - 3:B + 3] = (70, 0, 90, 64, 0, 65)
    lens[-1] = 100
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    m = H.make_model(binding, tabs, stack(g, (F, 1024, D)), stack(g, (D + T * (T + 1) // 2, 64, 1)), B, idx.size, F)
    m.set_option(binding.REC_OPT_STREAM_ROWS, int(stream))
    assert binding.rec_probe_plan_joined(m.handle, B, idx.size) == (binding.REC_OK, True)
    dense = g.standard_normal((B, F)).astype(np.float32)
    pooled = compare(binding, m, synth.Batch(dense, idx, lens))[4].cpu().numpy()
    H.check_pooled(pooled, *orc.pool(tabs, idx, lens, B, want_abs=True)[:2])
    bad = idx.copy()
    bad[[301, 700, idx.size - 2]] = (R, -1, R)
    H.run(m, synth.Batch(dense, bad, lens))
    assert m.check() == (binding.REC_ERR_INDEX_RANGE, 301)
    H.check_pooled(m.debug_pooled().cpu().numpy(), *orc.pool(tabs, bad, lens, B, want_abs=True)[:2])
    H.run(m, synth.Batch(dense, idx[:-3], lens))
    assert m.check() == (binding.REC_ERR_LENGTHS, -1)
    for at, v, first in ((n - 2, -7, n - 2), (5, -1, 5), (6, 1 << 20, -1), (700, (1 << 31) - 1, -1)):
        odd = lens.copy()
        odd[at] = v
        H.run(m, synth.Batch(dense, idx, odd))
        assert m.check() == (binding.REC_ERR_LENGTHS, first)
        off = np.minimum(orc.offsets(odd)[0], idx.size)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
    H.run(m, synth.Batch(dense, idx, lens))
    assert m.check() == (binding.REC_OK, -1) and np.array_equal(m.debug_pooled().cpu().numpy(), pooled)
    m.close()


def test_long_bags_in_every_eighth_four(binding):
    """No wave of a pooling block has its long bags to itself: fours that do not fit are dealt to all waves (when a
    block's waves took every eighth four the joint launch was 1.3 times as long as separate ones, now it is 0.7)."""
    print("beside wide, long bags", flush=True)
    g = np.random.default_rng(8)
    T, D, B, F, R = 10, 32, 4096, 1536, 400
    n = T * B
    tabs = [g.uniform(-1, 1, (R, D)).astype(np.float32) for _ in range(T)]
    lens = np.where(np.arange(n) % 32 < 4, 300, 2).astype(np.int32)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    m = H.make_model(binding, tabs, stack(g, (F, 1024, D)), stack(g, (D + T * (T + 1) // 2, 64, 1)), B, idx.size, F)
    assert binding.rec_probe_plan_joined(m.handle, B, idx.size) == (binding.REC_OK, True)
    dense = g.standard_normal((B, F)).astype(np.float32)
    H.run(m, synth.Batch(dense, idx, lens))
    assert m.check() == (binding.REC_OK, -1)
    H.check_pooled(m.debug_pooled().cpu().numpy(), *orc.pool(tabs, idx, lens, B, want_abs=True)[:2])
    args = [torch.from_numpy(a).cuda() for a in (dense, idx, lens)]
    out, best = torch.empty(B, device="cuda"), {}
    for fuse in (1, 0, 1, 0):
        m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                m.forward(*args, out)
            b.record()
            b.synchronize()
            best[fuse] = min(best.get(fuse, 1e9), a.elapsed_time(b) / 10)
    print(best, flush=True)
    assert best[1] <= 1.2 * best[0], best
    m.close()
