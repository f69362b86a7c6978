"""Two bags of a table by one wave: every row size that takes it, an odd and an even number of samples,
pairs whose ids just fit and do not, empty bags, faults; in blocks of one wave and (pipelined) of eight and, of
many more bags, four."""
import numpy as np
import pytest
import torch

from oracle import rec_oracle as orc
from paper_2203_07424_amd import synth

import gpu_helpers as H
from test_gpu_front import stack
from test_gpu_pool_fold import sums_in_order

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2203_07424_amd import binding as b
    return b


ROWS = [(64, np.float16, 0), (64, np.float32, 1), (128, np.float16, 1), (128, np.float32, 0), (256, np.float16, 0), (256, np.float32, 1)]


@pytest.mark.parametrize("rowbytes,dtype,odd,pipeline,rounds", [(*r, p, 5) for r in ROWS for p in (False, True)] + [(64, np.float32, 1, True, 64)])
def test_two_bags_by_a_wave(binding, rowbytes, dtype, odd, pipeline, rounds):
    print("two bags", rowbytes, np.dtype(dtype).name, odd, pipeline, rounds, flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    D, T, R, F = rowbytes // np.dtype(dtype).itemsize, 2, 300, 6
    B = (rounds * 32 * cus + T - 1) // T  # 5: the smallest batch, of bags of up to 2 KB of rows
    B += B % 2 != odd
    g = np.random.default_rng(300 + rowbytes + odd)
    # magnitudes over eight octaves, so that the order of a sum shows in fp16 rows as well
    tabs = [(g.uniform(-1, 1, (R, D)) * 2.0 ** g.integers(-8, 1, (R, D))).astype(dtype) for _ in range(T)]
    lens = g.integers(0, 13, T * B).astype(np.int32)
    # pairs of 256 and 257 ids, one bag of all of them, lengths around a wave-wide load's rows, the ends of a table
    lens[:16] = (128, 128, 128, 129, 256, 0, 0, 257, 1, 7, 8, 9, 31, 32, 33, 63)
    lens[B - 3:B + 3] = (70, 0, 90, 64, 0, 65)
    lens[-1] = 100
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    m = binding.RecModel(T, D, [R] * T, "f16" if dtype == np.float16 else "f32", F, [F, D], [D + 3, 1], B, idx.size, pipeline=pipeline)
    for t, tab in enumerate(tabs):
        m.load_table(t, torch.from_numpy(tab).cuda())
    assert cus != 256 or binding.rec_probe_plan_pooling(m.handle, B, idx.size) == (binding.REC_OK, binding.REC_POOL_TWO)
    H.load_mlps(binding, m, stack(g, (F, D)), stack(g, (D + 3, 1)))
    dense = g.standard_normal((B, F)).astype(np.float32)
    H.run(m, synth.Batch(dense, idx, lens))
    assert m.check() == (binding.REC_OK, -1)
    got = m.debug_pooled().cpu().numpy()
    P, A, _, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
    H.check_pooled(got, P, A)
    ends = np.cumsum(lens)
    for k in [*range(40), *range(B - 6, B + 6), *range(T * B - 6, T * B), *g.integers(0, T * B, 200)]:
        want = sums_in_order(tabs[k // B], idx[ends[k] - lens[k]:ends[k]], rowbytes // 16)
        assert np.array_equal(got[k % B, k // B], want), k
    bad = idx.copy()
    bad[[700, idx.size - 2]] = (R, -1)  # in a pair of the first table, and in the last bag
    H.run(m, synth.Batch(dense, bad, lens))
    assert m.check() == (binding.REC_ERR_INDEX_RANGE, 700)
    H.check_pooled(m.debug_pooled().cpu().numpy(), *orc.pool(tabs, bad, lens, B, want_abs=True)[:2])
    m.close()
