"""Interaction and Predict-FC (and the end of Bottom-FC) in one launch, at the sizes
where it can go wrong: the samples a block takes (8, 16 or 32) and one more than
whole blocks, 16-row blocks of the interaction, Predict-FC inputs wider than 1024,
layers of 1 to 4 chunks a wave.

Against the oracle's bars, and against the same model layer by layer: both narrow
the same operands to bf16 and differ in the order of fp32 sums only, which moves
a sum across a rounding boundary now and then (1e-3 for 98 % of the samples, 2e-2
for all, as for chains)."""
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


def close(a, b, scale):
    gap = np.abs(a.astype(np.float64) - b) / scale
    assert gap.max() <= 2e-2 and np.quantile(gap, 0.98) <= 1e-3, (gap.max(), np.quantile(gap, 0.98))


@pytest.mark.parametrize("T,D,B,F,hb,ht", [
    (2, 32, 1, 13, (40,), (24,)),
    (15, 64, 9, 8, (), (64, 33)),                 # dense input as given; V = 16
    (16, 32, 7, 20, (64,), (200, 72)),            # V = 17
    (47, 64, 2049, 30, (96,), (100, 50)),         # V = 48; 16 samples a block, one in the last
    (50, 64, 40, 30, (300,), (520, 300)),         # 1339 wide input
    (62, 64, 33, 16, (64,), (1024,)),             # V = 63, 2017 wide input, four chunks a wave
    (3, 32, 4097, 1500, (1100, 200), (700, 64)),  # Bottom-FC's last layers in the launch; 32 samples a block
    (4, 64, 300, 2000, (1100, 1000, 70), (96,)),
    (20, 64, 17, 30, (96,), (200, 72)),           # V = 21
    (31, 64, 300, 30, (), (512, 128)),            # V = 32
    (33, 32, 33, 30, (96,), (100, 50)),           # V = 34
    (47, 32, 2100, 30, (300,), (640, 64)),        # V = 48
    (49, 32, 25, 30, (96,), (256, 40)),           # V = 50
    (62, 32, 130, 30, (), (800, 300)),            # V = 63, 1985 wide input
])
def test_tail_in_one_launch(binding, T, D, B, F, hb, ht):
    print("tail case", T, D, B, F, hb, ht, flush=True)
    g = np.random.default_rng(800 + T + B)
    R = 60
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    lens = g.integers(0, 7, T * B).astype(np.int32)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    if not hb:
        F = D
    bottom = stack(g, (F,) + tuple(hb) + (D,)) if hb else []
    top = stack(g, (D + T * (T + 1) // 2,) + tuple(ht) + (1,))
    m = H.make_model(binding, tabs, bottom, top, B + 3, max(idx.size, 1), F)
    batch = synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, lens)
    m.set_option(binding.REC_OPT_FUSE_MLP, 0)
    plain = H.run(m, batch)
    z = m.debug_interact().clone()
    m.set_option(binding.REC_OPT_FUSE_MLP, 2)
    fused = H.run(m, batch)
    assert m.check() == (binding.REC_OK, -1)
    if len(hb) < 2:  # the same x0, so the same interaction: same products, same bits
        assert torch.equal(z.view(torch.int16), m.debug_interact().view(torch.int16))
    exact = orc.forward(batch.dense, tabs, idx, lens, bottom, top)["logits"]
    if B >= 8:
        H.check_logits(fused, exact)
    close(fused, plain, np.maximum(np.abs(exact), np.sqrt((exact ** 2).mean())))
    assert np.array_equal(fused, H.run(m, batch))
    m.close()


@pytest.mark.parametrize("hidden,per_cu,one", [
    ((512, 128), 1, False), ((512, 128), 12, True), ((1024, 128), 12, False), ((1024,) * 5, 12, False),
    ((1024,) * 5, 16, False), ((1024, 1024), 17, True), ((1024,) * 5, 32, False), ((512, 128), 33, False)])
def test_the_joint_launch_is_taken_by_weights_and_batch(binding, hidden, per_cu, one):
    """Left to itself the library takes the one launch where it is the faster: every
    block streams all weights, so heavy stacks stay layer by layer."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T, D, B, F, R = 40, 64, per_cu * cus, 20, 50
    print("tail rule", hidden, B, flush=True)
    g = np.random.default_rng(850)
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    bottom, top = stack(g, (F, 64, D)), stack(g, (D + T * (T + 1) // 2,) + hidden + (1,))
    m = H.make_model(binding, tabs, bottom, top, B, T * B, F)
    idx = g.integers(0, R, T * B).astype(np.int32)
    d = [torch.from_numpy(a).cuda() for a in (g.standard_normal((B, F)).astype(np.float32), idx, np.ones(T * B, np.int32))]
    m.set_profiling(1, 1)
    m.forward(*d)
    torch.cuda.synchronize()
    assert m.check() == (binding.REC_OK, -1)
    assert ("interact" in m.stage_shared(0)) == one
    m.set_profiling(0)
    m.close()
