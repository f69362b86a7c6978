"""Scan, dense part and lookups of a concatenation model in one launch of few large blocks: from the smallest
batch that takes it to the largest, row sizes, a batch and bags that are no multiple of a block, and lengths
that its quick sum in 32 bits is not for."""
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


@pytest.mark.parametrize("T,D,dtype,B,F", [(1, 64, np.float16, 12289, 7), (7, 32, np.float16, 1757, 64), (5, 32, np.float32, 9800, 20),
                                           (26, 64, np.float16, 5041, 24), (13, 64, np.float32, 5041, 5), (3, 16, np.float32, 43690, 12)])
def test_front_of_many_lookups(binding, T, D, dtype, B, F):
    print("front lookup case", T, D, np.dtype(dtype).name, B, F, flush=True)
    g = np.random.default_rng(960 + T + B)
    R, n = 300, T * B
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(dtype) for _ in range(T)]
    m = H.make_model(binding, tabs, [], stack(g, (F + T * D, 1)), B, 2 * n, F, interaction="concat")
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert binding.rec_probe_plan_pooling(m.handle, B, n) == (binding.REC_OK, binding.REC_POOL_MANY_LOOKUPS)
    dense = g.standard_normal((B, F)).astype(np.float32)

    def run(lens, idx):
        H.run(m, synth.Batch(dense, idx, lens))
        off = np.minimum(orc.offsets(lens)[0], idx.size)
        assert np.array_equal(m.debug_offsets().cpu().numpy().astype(np.int64), off)
        return m.debug_interact()

    ones, few = np.ones(n, np.int32), g.integers(0, 3, n).astype(np.int32)
    few[g.integers(0, n, 5)] = 9
    for lens in (ones, few):
        idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
        z = run(lens, idx)
        assert m.check() == (binding.REC_OK, -1)
        assert torch.equal(z[:, :F].cpu(), torch.from_numpy(dense).bfloat16()) and not z[:, F + T * D:].any()
        together = z.clone()
        m.set_option(binding.REC_OPT_FUSE_MLP, 0)  # scan and lookups as launches of their own
        assert torch.equal(run(lens, idx), together)
        m.set_option(binding.REC_OPT_FUSE_MLP, 1)
        P, A, _, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
        z = together[:, F:F + T * D].float().cpu().numpy().astype(np.float64).reshape(B, T, D)
        # half an ulp of bf16's 8 significant bits on a sum good to 1e-5 of the absolute sum
        assert (np.abs(z - P) <= 2.0 ** -8 * (np.abs(P) + 1e-5 * A) + 1e-5 * A).all()
    bad = idx.copy()
    bad[[9000, -1]] = (R, -1)
    run(few, bad)
    assert m.check() == (binding.REC_ERR_INDEX_RANGE, 9000)
    run(few, idx[:-3])
    assert m.check() == (binding.REC_ERR_LENGTHS, -1)
    for at, v, first in ((n - 2, -7, n - 2), (5, -1, 5), (6, 1 << 20, -1), (700, (1 << 31) - 1, -1)):
        odd = few.copy()
        odd[at] = v
        run(odd, idx)
        assert m.check() == (binding.REC_ERR_LENGTHS, first)
    m.close()


def test_long_bags(binding):
    """Bags of more ids than most: one that is nearly all of the forward takes no longer than in a launch of
    lookups alone (with an id at a time it took 1.8 times as long, with four 0.5), and every length around the ids of
    a trip gives the same sums; an id out of range in a late trip is found."""
    print("front lookup long bags", flush=True)
    g = np.random.default_rng(5)
    T, D, B, R, F = 26, 64, 600, 300, 8
    tabs = [g.uniform(-0.05, 0.05, (R, D)).astype(np.float16) for _ in range(T)]
    n = T * B
    lens = np.where(g.random(n) < 0.03, g.integers(0, 12, n), 1).astype(np.int32)
    lens[512:700], lens[5000:5100] = 6, 3
    lens[n // 3] = 0
    lens[n // 3] = n + n // 4 - lens.sum()
    assert lens[n // 3] > 400
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    m = H.make_model(binding, tabs, [], stack(g, (F + T * D, 1)), B, idx.size, F, interaction="concat")
    assert binding.rec_probe_plan(m.handle, B, idx.size)[1] & binding.REC_PLAN_FRONT
    dense = g.standard_normal((B, F)).astype(np.float32)
    H.run(m, synth.Batch(dense, idx, lens))
    assert m.check() == (binding.REC_OK, -1)
    z = m.debug_interact()[:, F:F + T * D].float().cpu().numpy().astype(np.float64).reshape(B, T, D)
    P, A, _, _ = orc.pool(tabs, idx, lens, B, want_abs=True)
    assert (np.abs(z - P) <= 2.0 ** -8 * (np.abs(P) + 1e-5 * A) + 1e-5 * A).all()
    bad, at = idx.copy(), int(lens[:n // 3 + 1].sum()) - 2
    bad[at] = R
    H.run(m, synth.Batch(dense, bad, lens))
    assert m.check() == (binding.REC_ERR_INDEX_RANGE, at)

    lens = np.ones(n, np.int32)
    lens[n // 3] = 3500
    idx = g.integers(0, R, int(lens.sum())).astype(np.int32)
    args = [torch.from_numpy(a).cuda() for a in (dense, idx, lens)]
    out, best = torch.empty(B, device="cuda"), {}
    for fuse in (1, 0, 1, 0):
        m.set_option(binding.REC_OPT_FUSE_MLP, fuse)
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                m.forward(*args, out)
            b.record()
            b.synchronize()
            best[fuse] = min(best.get(fuse, 1e9), a.elapsed_time(b))
    assert best[1] <= 1.2 * best[0], best
    m.close()
