"""The cross-lane fold of the pooling kernel for every row size it is compiled for
(16 bytes to 1 KB, fp16 and fp32 rows), into the fp32 buffer and, narrowed, into
the Predict-FC input of a concatenation model (aligned and unaligned columns)."""
import numpy as np
import pytest

from oracle import rec_oracle as orc
from paper_2203_07424_amd import synth

import gpu_helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2203_07424_amd import binding as b
    return b


@pytest.mark.parametrize("interaction,F", [("dot", 6), ("concat", 8), ("concat", 5)])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("rowbytes", [16, 32, 64, 128, 256, 512, 1024])
def test_fold_of_every_row_size(binding, rowbytes, dtype, interaction, F):
    print("fold case", rowbytes, np.dtype(dtype).name, interaction, F, flush=True)
    D = rowbytes // np.dtype(dtype).itemsize
    T, R, B = 2, 90, 21
    g = np.random.default_rng(40 + rowbytes + F)
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    lens = g.integers(0, 150, T * B).astype(np.int32)
    lens[:3] = (0, 1, 64)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    layer = lambda n, k: [((g.standard_normal((n, k)) * k ** -0.5).astype(np.float32), np.zeros(n, np.float32))]
    dot = interaction == "dot"
    bottom = layer(D, F) if dot else []
    width = D + T * (T + 1) // 2 if dot else F + T * D
    m = H.make_model(binding, tabs, bottom, layer(1, width), B, idx.size, F, interaction=interaction)
    H.run(m, synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, lens))
    assert m.check() == (binding.REC_OK, -1)
    P, A, nbad, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
    assert nbad == 0
    if dot:
        H.check_pooled(m.debug_pooled().cpu().numpy(), P, A)
    else:  # half an ulp of bf16's 8 significant bits (2^-8 of the value) on a sum good to 1e-5 of the absolute sum
        z = m.debug_interact().float().cpu().numpy().astype(np.float64)[:, F:F + T * D].reshape(B, T, D)
        assert (np.abs(z - P) <= 2.0 ** -8 * (np.abs(P) + 1e-5 * A) + 1e-5 * A + 1e-30).all()
    m.close()


def sums_in_order(tab, ids, lpr):
    """The sum of a bag in fp32 as the pooling wave takes it: row j of the bag goes to
    partial sum j % RPW in the order of the bag (64 ids at a time, a multiple of RPW),
    then the partial sums are folded r with r ^ 1, r ^ 2, r ^ 4, ..."""
    rpw = 64 // lpr
    part = np.zeros((rpw, tab.shape[1]), np.float32)
    for j, i in enumerate(ids):
        part[j % rpw] += tab[i].astype(np.float32)
    while part.shape[0] > 1:
        part = part[0::2] + part[1::2]
    return part[0]


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("rowbytes", [16, 32, 64, 128, 256, 512, 1024])
def test_sums_are_taken_in_the_stated_order(binding, rowbytes, dtype):
    """Bit for bit: fp32 sums in another order differ in their last bits, and these
    change which way a term of the interaction is rounded to bf16."""
    print("fold order", rowbytes, np.dtype(dtype).name, flush=True)
    D = rowbytes // np.dtype(dtype).itemsize
    T, R, B, F = 2, 90, 21, 6
    g = np.random.default_rng(70 + rowbytes)
    # magnitudes over eight octaves, so that the order of a sum shows in fp16 rows as well
    tabs = [(g.uniform(-1, 1, (R, D)) * 2.0 ** g.integers(-8, 1, (R, D))).astype(dtype) for _ in range(T)]
    lens = g.integers(5, 150, T * B).astype(np.int32)
    lens[:3] = (0, 1, 64)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    layer = lambda n, k: [((g.standard_normal((n, k)) * k ** -0.5).astype(np.float32), np.zeros(n, np.float32))]
    m = H.make_model(binding, tabs, layer(D, F), layer(1, D + T * (T + 1) // 2), B, idx.size, F)
    H.run(m, synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, lens))
    assert m.check() == (binding.REC_OK, -1)
    got = m.debug_pooled().cpu().numpy()
    ends = np.cumsum(lens)
    for t in range(T):
        for b in range(B):
            k = t * B + b
            want = sums_in_order(tabs[t], idx[ends[k] - lens[k]:ends[k]], rowbytes // 16)
            assert np.array_equal(got[b, t], want), (t, b)
    m.close()
