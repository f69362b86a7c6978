"""Scan, Bottom-FC and pooling in one launch where Bottom-FC keeps within 64 registers: from the
smallest batch that takes this form by its bags to the largest and one bag more, a Bottom-FC
of one to three layers, the widest input."""
import numpy as np
import pytest
import torch

from oracle import rec_oracle as orc
from paper_2203_07424_amd import synth

import gpu_helpers as H
from test_gpu_front import stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2203_07424_amd import binding as b
    return b


@pytest.mark.parametrize("T,D,dtype,B,bottom", [(7, 64, np.float16, 1025, (30, 64)), (23, 32, np.float32, 312, (512, 256, 32)),
                                                (8, 64, np.float16, 1792, (13, 256, 128, 64)), (3, 64, np.float32, 4779, (257, 100, 64)),
                                                (10, 16, np.float32, 1003, (500, 16))])
def test_front_of_more_bags(binding, T, D, dtype, B, bottom):
    print("front light case", T, D, np.dtype(dtype).name, B, bottom, flush=True)
    g = np.random.default_rng(700 + T + B)
    R, F = 500, bottom[0]
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    lens = g.integers(0, 16, T * B).astype(np.int32)
    lens[-1] = 131
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    m = H.make_model(binding, tabs, stack(g, bottom), stack(g, (D + T * (T + 1) // 2, 1)), B, idx.size, F)
    dense = g.standard_normal((B, F)).astype(np.float32)
    for l, i in ((lens, idx), (lens, idx[:-70])):  # as stated, and too few ids: bags cut off at their number
        H.run(m, synth.Batch(dense, i, l))
        assert m.check() == ((binding.REC_OK, -1) if i is idx else (binding.REC_ERR_LENGTHS, -1))
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), np.minimum(orc.offsets(l)[0], i.size))
        pooled, x0 = m.debug_pooled().clone(), m.debug_bottom_out().clone()
        m.set_option(binding.REC_OPT_OVERLAP_DENSE, 1)  # scan, pooling and Bottom-FC as launches of their own
        H.run(m, synth.Batch(dense, i, l))
        m.check()
        assert torch.equal(pooled, m.debug_pooled()) and torch.equal(x0, m.debug_bottom_out())
        m.set_option(binding.REC_OPT_OVERLAP_DENSE, 0)
    m.close()
