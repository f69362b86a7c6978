"""Scan, Bottom-FC and pooling in one launch (batches of up to
6144 bags, 12288 of a few ids), at the
edges of its blocks: 8 bags a block of the pooled form, 32 to 128 of the short-bag
form, scan tiles of 2048, the largest batch it takes and one bag more.

Pooled sums and Bottom-FC against the same kernels' bodies in launches of their
own (same bits), offsets against the oracle (exact), faults as ever."""
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


@pytest.mark.parametrize("T,D,dtype,B", [(1, 32, np.float16, 1), (7, 64, np.float16, 1), (3, 32, np.float32, 3),
                                         (23, 64, np.float32, 89), (16, 64, np.float16, 128), (3, 32, np.float16, 683),
                                         (8, 64, np.float16, 768), (5, 32, np.float32, 1229), (29, 64, np.float16, 565),
                                         (6, 16, np.float32, 130), (9, 128, np.float16, 75)])
def test_front_of_pooled_models(binding, T, D, dtype, B):
    print("front case", T, D, np.dtype(dtype).name, B, flush=True)
    g = np.random.default_rng(900 + T + B)
    R, F = 400, 30
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    lens = g.integers(0, 30, T * B).astype(np.int32)
    lens[0] = 67
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    m = H.make_model(binding, tabs, stack(g, (F, 70, D)), stack(g, (D + T * (T + 1) // 2, 1)), B, idx.size, F)
    dense = g.standard_normal((B, F)).astype(np.float32)
    batch = synth.Batch(dense, idx, lens)
    H.run(m, batch)
    assert m.check() == (binding.REC_OK, -1)
    off, _, _ = orc.offsets(lens)
    assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
    pooled, x0 = m.debug_pooled().clone(), m.debug_bottom_out().clone()
    P, A, _, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
    H.check_pooled(pooled.cpu().numpy(), P, A)
    m.set_option(binding.REC_OPT_OVERLAP_DENSE, 1)   # scan, pooling and Bottom-FC as launches of their own
    H.run(m, batch)
    assert torch.equal(pooled, m.debug_pooled()) and torch.equal(x0, m.debug_bottom_out())
    m.set_option(binding.REC_OPT_OVERLAP_DENSE, 0)
    m.set_option(binding.REC_OPT_STREAM_ROWS, 1)
    H.run(m, batch)
    assert torch.equal(pooled, m.debug_pooled())
    # faults: a negative length near the end, ids outside the table, too few ids
    if T * B > 20:
        neg = lens.copy()
        at = neg.size - 9
        cut, start = int(neg[at]), int(lens[:at].sum())
        neg[at] = -cut - 3
        H.run(m, synth.Batch(dense, np.concatenate([idx[:start], idx[start + cut:]]), neg))
        off, _, _ = orc.offsets(neg)
        assert m.check() == (binding.REC_ERR_LENGTHS, at)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
        bad = idx.copy()
        bad[[5, idx.size - 2]] = (R, -1)
        H.run(m, synth.Batch(dense, bad, lens))
        assert m.check() == (binding.REC_ERR_INDEX_RANGE, 5)
        H.check_pooled(m.debug_pooled().cpu().numpy(), *orc.pool(tabs, bad, lens, B, want_abs=True)[:2])
        H.run(m, synth.Batch(dense, idx[:-70], lens))
        assert m.check() == (binding.REC_ERR_LENGTHS, -1)
        assert int(m.debug_offsets().max()) == idx.size - 70
        H.run(m, batch)
        assert m.check() == (binding.REC_OK, -1) and torch.equal(pooled, m.debug_pooled())
    m.close()


@pytest.mark.parametrize("T,D,dtype,B,F", [(1, 32, np.float16, 1, 8), (3, 64, np.float16, 43, 24), (5, 32, np.float16, 77, 5),
                                           (7, 64, np.float32, 293, 20), (26, 64, np.float16, 300, 64),
                                           (4, 32, np.float32, 3072, 16), (1, 64, np.float16, 12289, 7),
                                           (6, 16, np.float32, 55, 12), (5, 128, np.float16, 31, 16)])
def test_front_of_concatenation_models(binding, T, D, dtype, B, F):
    print("front concat case", T, D, np.dtype(dtype).name, B, F, flush=True)
    g = np.random.default_rng(930 + T + B)
    R = 300
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    m = H.make_model(binding, tabs, [], stack(g, (F + T * D, 1)), B, 4 * T * B, F, interaction="concat")
    dense = g.standard_normal((B, F)).astype(np.float32)
    for lens in (np.ones(T * B, np.int32), g.integers(0, 4, T * B).astype(np.int32)):
        lens[0] = max(int(lens[0]), 1)
        idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
        H.run(m, synth.Batch(dense, idx, lens))
        assert m.check() == (binding.REC_OK, -1)
        off, _, _ = orc.offsets(lens)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
        z = m.debug_interact()
        assert torch.equal(z[:, :F].cpu(), torch.from_numpy(dense).bfloat16()) and not z[:, F + T * D:].any()
        z = z[:, F:F + T * D].float().cpu().numpy().astype(np.float64).reshape(B, T, D)
        P, A, _, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
        # half an ulp of bf16's 8 significant bits on a sum good to 1e-5 of the absolute sum
        assert (np.abs(z - P) <= 2.0 ** -8 * (np.abs(P) + 1e-5 * A) + 1e-5 * A).all()
    bad = idx.copy()
    bad[-1] = R
    H.run(m, synth.Batch(dense, bad, lens))
    assert m.check() == (binding.REC_ERR_INDEX_RANGE, idx.size - 1)
    if T * B > 50:
        neg = lens.copy()
        neg[40], lost = -2, int(lens[40])
        start = int(lens[:40].sum())
        H.run(m, synth.Batch(dense, np.concatenate([idx[:start], idx[start + lost:]]), neg))
        assert m.check() == (binding.REC_ERR_LENGTHS, 40)
    m.close()
