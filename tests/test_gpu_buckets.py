"""Sums of gradient buckets on the GPU at the sizes where their reduction changes: a thread per leaf, a wave per leaf
(one to several batches of rows), a wave for every leaf of a small tree; dense gradients and both fused optimisers."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2307_15333_amd import core, synth

from .test_gpu_backward import GTOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("small", [True, False])
def test_bucket_sizes(degree, small):
    """n copies of one ray put n equal rows into each bucket it meets: the gradient is n times the ray's, within the
    usual 1e-4 of the largest value (the sums round n 2^-24 at most, 4e-5 here) and what the FP32 prefix sums of a
    segment allow (sqrt(3) |g|_1 (N + 4) 2^-23 for each of n rays of N segments).  A fused step applies the formula of
    the separate step to the same sums: they differ by a few roundings of it."""
    s = synth.uniform_scene(1, degree, 0.8, seed=degree) if small else synth.random_tree_scene(5, degree, seed=90 + degree, p_split=0.5)
    ref = O.OracleTree.from_scene(s, sigma=s.sigma.astype(np.float64))
    o, d = synth.random_explicit_rays(1, seed=7)
    g = np.array([[0.7, -0.4, 1.1]], np.float32)
    rs, rh = O.backward(ref, o.astype(np.float64), d.astype(np.float64), g.astype(np.float64), t_stop=0.0)
    assert (rs != 0).any()
    for n in (1, 31, 32, 33, 64, 65, 128, 129, 256, 257, 700):
        tree = core.Octree.from_scene(s)
        rays = core.Rays.explicit(np.repeat(o, n, 0), np.repeat(d, n, 0))
        gg = torch.as_tensor(np.repeat(g, n, 0), device="cuda")
        rec = torch.empty(core.Octree.records_bytes(n, 64), dtype=torch.uint8, device="cuda")
        rgb, ns, cnt = tree.render_train(rays, t_stop=0.0, records=rec)
        kw = dict(t_stop=0.0, leaf_count=cnt, records=rec)
        gs = torch.zeros(tree.n_leaves, device="cuda")
        gh = torch.zeros((tree.n_leaves, 3, tree.K), device="cuda")
        tree.backward(rays, rgb, ns, gg, gs, gh, **kw)
        fp32 = np.sqrt(3.0) * np.abs(g).sum() * (int(ns.max()) + 4) * 2.0 ** -23
        assert np.abs(gs.cpu().numpy() / n - rs).max() <= GTOL * np.abs(rs).max() + fp32
        assert np.abs(gh.cpu().numpy() / n - rh).max() <= GTOL * np.abs(rh).max()
        for kind in ("rmsprop", "adam"):
            a, b = core.Octree.from_scene(s), core.Octree.from_scene(s)
            if kind == "rmsprop":
                a.rmsprop_step(gs, gh, a.rmsprop_state(), eps=1e-4)
                b.backward_rmsprop(rays, rgb, ns, gg, b.rmsprop_state(), eps=1e-4, **kw)
            else:
                a.adam_step(gs, gh, a.adam_state(), 1, eps=1e-4)
                b.backward_adam(rays, rgb, ns, gg, b.adam_state(), 1, eps=1e-4, **kw)
            x, y = a.export(), b.export()
            np.testing.assert_allclose(y["sigma"], x["sigma"], rtol=1e-5, atol=1e-6)
            np.testing.assert_allclose(y["sh"], x["sh"], rtol=1e-5, atol=1e-6)
            a.close()
            b.close()
        tree.close()
