"""Interaction by one wave per sample, operands in registers, at the edges of its
16-row blocks and of the shapes it takes (D = 32 or 64, up to 63 tables), and
just past them, where the LDS-tiled kernel runs.

Each term against the oracle's formula on the device's own fp32 inputs: the bf16
narrowing of the output (2^-9 relative, 2^-8 allowed) plus a dot product good to
2^-16 of sum |x_i y_i| (2^-14 allowed), as in the whole-forward parity test."""
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


@pytest.mark.parametrize("T,D,B", [(1, 32, 1), (15, 32, 5), (16, 64, 9), (31, 64, 3), (32, 32, 130), (47, 64, 7),
                                   (48, 32, 4), (63, 64, 6), (63, 32, 3), (64, 32, 3), (4, 16, 11), (5, 128, 5)])
def test_interaction_terms_against_the_oracle_formula(binding, T, D, B):
    print("interaction case", T, D, B, flush=True)
    g = np.random.default_rng(700 + T + D + B)
    R, F = 50, 20
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float32) for _ in range(T)]
    lens = g.integers(0, 9, T * B).astype(np.int32)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    width = D + T * (T + 1) // 2
    layer = lambda n, k: [((g.standard_normal((n, k)) * k ** -0.5).astype(np.float32),
                           g.standard_normal(n).astype(np.float32) * 0.1)]
    m = H.make_model(binding, tabs, layer(D, F), layer(1, width), B, max(idx.size, 1), F)
    m.set_option(binding.REC_OPT_FUSE_MLP, 0)
    H.run(m, synth.Batch(g.standard_normal((B, F)).astype(np.float32), idx, lens))
    assert m.check() == (binding.REC_OK, -1)
    x0 = m.debug_bottom_out().cpu().numpy().astype(np.float64)
    P = m.debug_pooled().cpu().numpy().astype(np.float64)
    z = m.debug_interact().float().cpu().numpy().astype(np.float64)
    assert not z[:, width:].any()
    want, scale = orc.interact(x0, P), orc.interact(np.abs(x0), np.abs(P))
    scale[:, :D] = 0.0
    assert (np.abs(z[:, :width] - want) <= 2.0 ** -8 * np.abs(want) + 2.0 ** -14 * scale + 1e-30).all()
    m.close()
