"""FC layers with the k of a block tile dealt to the waves, at the edges of their
tiles: rows around 16, 32 and 64, the most and the fewest columns, one unit of 64 k
and more than the waves take at once, fp32 input rows aligned and not, the one-output
layer folded in for every width it is compiled for.

Against the same model layer by layer (REC_OPT_FUSE_MLP = 0, sums over k in order)
and against the oracle's bars.  Where only one layer lies between the input and
the compared value nothing is narrowed behind the sums, so the two device paths
differ by fp32 rounding only: K + log terms of at most 2^-24 of the sum of
magnitudes each, held to 2e-5 of the largest magnitude.  Behind several layers a
sum can cross a bf16 rounding boundary (1e-3 for 98 % of the samples, 2e-2 for all,
as for chains)."""
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


def stack(g, ws):
    return [((g.standard_normal((ws[i + 1], ws[i])) * ws[i] ** -0.5).astype(np.float32),
             (g.standard_normal(ws[i + 1]) * ws[i] ** -0.5).astype(np.float32))
            for i in range(len(ws) - 1)]


def close(a, b, scale):
    gap = np.abs(a.astype(np.float64) - b) / scale
    assert gap.max() <= 2e-2 and np.quantile(gap, 0.98) <= 1e-3, (gap.max(), np.quantile(gap, 0.98))


def both(binding, m, batch):
    m.set_option(binding.REC_OPT_FUSE_MLP, 0)
    plain = H.run(m, batch)
    m.set_option(binding.REC_OPT_FUSE_MLP, 1)
    got = H.run(m, batch)
    assert m.check() == (binding.REC_OK, -1)
    assert np.array_equal(got, H.run(m, batch))  # fixed order of sums
    return got, plain


TOWERS = [  # with the tiles of the layers on 256 compute units
    (1, 10, 64, 64, (512, 128), 1),            # 16 x 16, dot 16 x 128
    (16, 10, 64, 40, (512, 64), 3),            # 16 x 16, dot 16 x 64
    (17, 26, 64, 64, (1024, 512, 256), 4),     # 16 x 32, 16 x 16, dot 16 x 256
    (31, 12, 64, 10, (640, 256), 2),
    (65, 30, 64, 100, (1100, 1000, 72), 2),    # 32 x 32 twice, eight waves
    (300, 26, 64, 64, (1024, 512, 256), 4),    # 80 x 64, 48 x 64
    (200, 26, 64, 64, (1024, 512, 256), 4),    # 64 x 64 and 32 x 64, eight waves
    (320, 26, 64, 64, (1024, 512, 256), 4),    # 80 x 64, the last block full
    (257, 10, 64, 40, (1100, 1000, 72), 3),    # 32 x 64, four waves, 64 x 64, eight
    (300, 10, 64, 7, (448,), 8),               # the layer leaves fp32 for a dot kernel
    (1000, 20, 64, 33, (600, 200), 3),         # 64 x 64, four waves
    (520, 26, 64, 64, (1024, 512, 256), 4),    # 160 tiles of 128 x 128 instead, then one round of 80 rows
    (520, 3, 64, 64, (250, 1100), 1),          # 32 x 32, four waves
    (2100, 8, 64, 64, (256,), 4),              # dot 64 x 256
    (600, 8, 64, 64, (256,), 8),               # dot 32 x 256
    (2500, 4, 64, 64, (128,), 3),              # dot 32 x 128
]


@pytest.mark.parametrize("B,T,D,F,hidden,towers", TOWERS)
def test_towers_layer_by_layer(binding, B, T, D, F, hidden, towers):
    print("split towers", B, T, D, F, hidden, towers, flush=True)
    g = np.random.default_rng(1000 + B + T)
    R = 50
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    idx = g.integers(0, R, T * B).astype(np.int32)
    lens = np.ones(T * B, np.int32)
    tops = [stack(g, (F + T * D,) + hidden + (1,)) for _ in range(towers)]
    m = H.make_model(binding, tabs, [], tops, B, T * B, F, interaction="concat")
    batch = synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, lens)
    got, plain = both(binding, m, batch)
    exact = orc.forward_towers(batch.dense, tabs, idx, lens, [], tops, orc.EXACT)["logits"]
    got, plain, exact = (x.reshape(B, towers) for x in (got, plain, exact))
    for k in range(towers):
        if B >= 8:
            H.check_logits(got[:, k], exact[:, k])
        close(got[:, k], plain[:, k], np.maximum(np.abs(exact[:, k]), np.sqrt((exact[:, k] ** 2).mean())))
    m.close()


@pytest.mark.parametrize("N", [50, 64, 128, 256])
@pytest.mark.parametrize("B,towers", [(1, 1), (18, 3), (2100, 2), (2100, 4), (6200, 2)])
def test_one_layer_and_the_dot_behind_it(binding, N, B, towers):
    print("split dot", N, B, towers, flush=True)
    g = np.random.default_rng(1100 + N + B)
    T, D, F, R = 3, 64, 9, 40
    tabs = [g.uniform(-1, 1, (R, D)).astype(np.float16) for _ in range(T)]
    idx = g.integers(0, R, T * B).astype(np.int32)
    tops = [stack(g, (F + T * D, N, 1)) for _ in range(towers)]
    m = H.make_model(binding, tabs, [], tops, B, T * B, F, interaction="concat")
    got, plain = both(binding, m, synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, np.ones(T * B, np.int32)))
    assert np.abs(got.astype(np.float64) - plain).max() <= 2e-5 * max(np.abs(plain).max(), 1.0)
    m.close()


@pytest.mark.parametrize("B,F,D", [(1, 2560, 32), (33, 2560, 64), (300, 2560, 64), (600, 1000, 32), (5, 3, 8), (40, 4, 16),
                                   (70, 1501, 64), (1, 63, 32), (129, 66, 32)])
def test_dense_input_through_one_layer(binding, B, F, D):
    """fp32 rows, an fp32 result: the whole of a one-layer Bottom-FC."""
    print("split dense", B, F, D, flush=True)
    g = np.random.default_rng(1200 + B + F)
    T, R = 2, 30
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float32) for _ in range(T)]
    idx = g.integers(0, R, T * B).astype(np.int32)
    bottom, top = stack(g, (F, D)), stack(g, (D + T * (T + 1) // 2, 1))
    m = H.make_model(binding, tabs, bottom, top, B, T * B, F)
    batch = synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, np.ones(T * B, np.int32))
    x0 = []
    for fuse in (0, 1):
        m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
        H.run(m, batch)
        x0.append(m.debug_bottom_out().cpu().numpy()[:B].astype(np.float64))
    assert m.check() == (binding.REC_OK, -1)
    mirror = orc.forward(batch.dense, tabs, idx, batch.lengths, bottom, top, orc.BF16_MIRROR)["bottom_out"]
    assert np.abs(x0[1] - x0[0]).max() <= 2e-5 * max(np.abs(x0[0]).max(), 1.0)
    assert np.abs(x0[1][:, :D] - mirror).max() <= 2e-5 * max(np.abs(mirror).max(), 1.0)
    assert not x0[1][:, D:].any()
    m.close()


def test_dense_input_at_an_odd_address(binding):
    """Rows that start 4 bytes behind a 16-byte boundary take single loads."""
    import torch
    print("split dense, odd address", flush=True)
    g = np.random.default_rng(1300)
    T, D, F, B, R = 2, 32, 1200, 50, 30
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float32) for _ in range(T)]
    bottom, top = stack(g, (F, D)), stack(g, (D + 3, 1))
    m = H.make_model(binding, tabs, bottom, top, B, T * B, F)
    dense = g.standard_normal((B, F)).astype(np.float32)
    i, l = torch.from_numpy(g.integers(0, R, T * B).astype(np.int32)).cuda(), torch.ones(T * B, dtype=torch.int32, device="cuda")
    buf = torch.empty(B * F + 1, device="cuda")
    odd = buf[1:].view(B, F)
    odd.copy_(torch.from_numpy(dense))
    a, b = m.forward(torch.from_numpy(dense).cuda(), i, l), m.forward(odd, i, l)
    torch.cuda.synchronize()
    assert m.check() == (binding.REC_OK, -1) and torch.equal(a, b)
    m.close()
