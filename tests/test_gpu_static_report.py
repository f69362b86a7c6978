"""rec_forward_static()'s fault report from the launch that ends the forward: the joint
Predict-FC launch, a chain, the last layer with its dot, or (none of them) a launch of
its own; fewer blocks than compute units and more."""
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


@pytest.mark.parametrize("concat,hidden,towers,B,fuse", [
    (False, (64,), 1, 1, 1), (False, (64,), 1, 3000, 1),         # joint launch
    (True, (96, 72), 2, 50, 1), (True, (96, 72), 2, 2100, 1),    # chain
    (True, (512, 256), 2, 50, 1), (True, (512, 100), 1, 2100, 1),  # k dealt to waves, dot folded in
    (False, (64,), 1, 70, 0), (True, (50,), 2, 5000, 1), (True, (64,), 4, 4096, 1),  # k-tile by k-tile, dot folded in
    (True, (448,), 2, 70, 1), (True, (), 1, 33, 1)])  # a launch of its own
def test_faults_of_a_static_forward(binding, concat, hidden, towers, B, fuse):
    print("static report", concat, hidden, towers, B, fuse, flush=True)
    g = np.random.default_rng(1700 + B)
    T, D, F, R = 3, 32, 32 if not concat else 20, 60
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float32) for _ in range(T)]
    z = F + T * D if concat else D + T * (T + 1) // 2
    tops = [stack(g, (z,) + hidden + (1,)) for _ in range(towers)]
    m = H.make_model(binding, tabs, [], tops if concat else tops[0], B, 9 * T * B, F, interaction="concat" if concat else "dot")
    m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
    lens = g.integers(1, 3 if concat else 9, T * B).astype(np.int32)
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    dense = g.standard_normal((B, F)).astype(np.float32)
    want = torch.from_numpy(H.run(m, synth.Batch(dense, idx, lens)))
    out = torch.empty(want.shape, device="cuda")
    at = lens.size - 1
    neg, bad = lens.copy(), idx.copy()
    neg[at] = -4
    bad[idx.size - 1] = R
    first = int(lens[:at].sum())
    for i, l, report in ((idx, lens, (binding.REC_OK, -1)), (bad, lens, (binding.REC_ERR_INDEX_RANGE, idx.size - 1)),
                         (idx[:first], neg, (binding.REC_ERR_LENGTHS, at)), (idx[:-1], lens, (binding.REC_ERR_LENGTHS, -1)),
                         (idx, lens, (binding.REC_OK, -1))):
        fault = torch.full((2,), 77, dtype=torch.int64, device="cuda")
        args = [torch.from_numpy(a).cuda() for a in (dense, i, l)]
        m.forward_static(*args, out, fault)
        assert tuple(fault.tolist()) == report
        m.forward_static(*args, out, None)
    torch.cuda.synchronize()
    assert torch.equal(out.cpu(), want)
    m.close()
