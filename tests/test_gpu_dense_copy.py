"""The dense part of a concatenation model without Bottom-FC and the zeros behind each row, by the launches that
copy it (scan and a few lookups, scan alone, scan and many lookups): columns around the lanes of a wave and their
halves, rows around those of a unit."""
import numpy as np
import pytest
import torch

from paper_2203_07424_amd import synth

import gpu_helpers as H
from test_gpu_front import stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2203_07424_amd import binding as b
    return b


@pytest.mark.parametrize("F,T,B", [(1, 3, 1), (7, 3, 33), (7, 6, 2050), (24, 5, 129), (32, 2, 9), (33, 3, 6), (63, 7, 1757), (64, 3, 5), (65, 2, 3),
                                   (100, 26, 500), (1000, 26, 75), (1000, 26, 501), (2560, 26, 1), (2560, 7, 2047)])
def test_rows_and_zeros(binding, F, T, B):
    print("dense copy", F, T, B, flush=True)
    g = np.random.default_rng(40 + F + B)
    D, R = 32, 50
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float32) for _ in range(T)]
    m = H.make_model(binding, tabs, [], stack(g, (F + T * D, 1)), B, T * B, F, interaction="concat")
    idx, lens = g.integers(0, R, T * B).astype(np.int32), np.ones(T * B, np.int32)
    for fuse in (1, 0):  # 0: beyond a few lookups scan and lookups are launches of their own
        m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
        dense = g.standard_normal((B, F)).astype(np.float32)
        batch = synth.Batch(dense, idx, lens)
        H.run(m, batch)
        m.debug_interact().fill_(7.0)
        H.run(m, batch)
        z = m.debug_interact()
        assert torch.equal(z[:, :F].cpu(), torch.from_numpy(dense).bfloat16()) and not z[:, F + T * D:].any()
    m.close()
