"""Dense gradients where the reduction of the buckets changes its launches: few rows a leaf (heavy buckets in a launch
of their own) and more (in the light ones' launch), with and without heavy buckets, last workgroups that are nearly
empty; against the FP64 oracle with the bounds of the adjoint's other tests (1e-4 of the largest value, and
sqrt(3) |g|_1 (N + 4) 2^-23 for each of the rays in a leaf, whose N segments' FP32 prefix sums cancel)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2307_15333_amd import core, synth

from .test_gpu_backward import GTOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("depth,copies,spread", [(2, 20, 0), (2, 40, 0), (2, 70, 0), (2, 0, 300), (3, 40, 100),
                                                 (3, 400, 200), (3, 0, 40)])
def test_launches_of_the_reduction(degree, depth, copies, spread):
    s = synth.uniform_scene(depth, degree, 0.8, seed=degree)
    tree = core.Octree.from_scene(s)
    o1, d1 = synth.random_explicit_rays(1, seed=7)
    o2, d2 = synth.random_explicit_rays(max(spread, 1), seed=8)
    o = np.concatenate([np.repeat(o1, copies, 0), o2[:spread]])
    d = np.concatenate([np.repeat(d1, copies, 0), d2[:spread]])
    n = copies + spread
    g = np.random.default_rng(n).normal(size=(n, 3)).astype(np.float32)
    rays = core.Rays.explicit(o, d)
    rs, rh = O.backward(O.OracleTree.from_scene(s, sigma=s.sigma.astype(np.float64)), o.astype(np.float64),
                        d.astype(np.float64), g.astype(np.float64), t_stop=0.0)
    gg = torch.as_tensor(g, device="cuda")
    for records in (64, 5, None):
        cnt = rec = None
        if records:
            rec = torch.empty(core.Octree.records_bytes(n, records), dtype=torch.uint8, device="cuda")
            rgb, ns, cnt = tree.render_train(rays, t_stop=0.0, records=rec)
        else:
            rgb, ns = tree.render(rays, t_stop=0.0, nseg=True)
        # added to what is there
        gs = torch.ones(tree.n_leaves, device="cuda")
        gh = torch.ones((tree.n_leaves, 3, tree.K), device="cuda")
        tree.backward(rays, rgb, ns, gg, gs, gh, t_stop=0.0, leaf_count=cnt, records=rec)
        fp32 = np.sqrt(3.0) * (np.abs(g).sum(1) * (ns.cpu().numpy() + 4)).sum() * 2.0 ** -23 + n * 2.0 ** -24
        assert np.abs(gs.cpu().numpy() - 1.0 - rs).max() <= GTOL * np.abs(rs).max() + fp32
        assert np.abs(gh.cpu().numpy() - 1.0 - rh).max() <= GTOL * np.abs(rh).max() + n * 2.0 ** -24
