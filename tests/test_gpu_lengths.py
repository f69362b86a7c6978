"""Launches whose blocks add up all earlier lengths themselves: lengths that start
on a 16-byte boundary and 4, 8 and 12 bytes behind one give the same offsets and the
same logits, negative lengths count as zero on either path."""
import numpy as np
import pytest
import torch

from oracle import rec_oracle as orc

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


@pytest.mark.parametrize("T,B,concat", [(1, 1, False), (1, 3, False), (3, 7, False), (8, 37, False), (12, 512, False),
                                        (13, 1000, False), (26, 300, True), (5, 13, True), (1, 2, True), (24, 512, True)])
def test_lengths_at_any_address(binding, T, B, concat):
    print("lengths", T, B, concat, flush=True)
    g = np.random.default_rng(1400 + T * B)
    R, D, F = 60, 64, 12
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    lens = g.integers(0, 3 if concat else 12, T * B).astype(np.int32)
    if not concat:
        lens[0] = 6 * T * B  # mean above what the short-bag form takes
    for k in (1, T * B // 2):
        if k < T * B - 1:
            lens[k] = -3
    off, _, _ = orc.offsets(lens)
    nnz = int(np.maximum(lens, 0).sum())
    idx = g.integers(0, R, max(nnz, 1)).astype(np.int32)[:nnz]
    if concat:
        m = H.make_model(binding, tabs, [], stack(g, (F + T * D, 40, 1)), B, nnz, F, interaction="concat")
    else:
        m = H.make_model(binding, tabs, stack(g, (F, 70, D)), stack(g, (D + T * (T + 1) // 2, 40, 1)), B, nnz, F)
    dense, ids = (torch.from_numpy(a).cuda() for a in (g.standard_normal((B, F)).astype(np.float32), idx))
    buf = torch.empty(T * B + 3, dtype=torch.int32, device="cuda")
    first = None
    for shift in range(4):
        at = buf[shift:shift + T * B]
        at.copy_(torch.from_numpy(lens))
        got = m.forward(dense, ids, at)
        torch.cuda.synchronize()
        st, _ = m.check()
        assert st == (binding.REC_ERR_LENGTHS if (lens < 0).any() else binding.REC_OK)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
        first = got.clone() if first is None else first
        assert torch.equal(got, first), shift
    m.close()
