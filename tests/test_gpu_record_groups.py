"""Records of a training forward lie in groups of four slots, the last one of what is left: capacities of a whole group
and a part of one, on rays of fewer, as many and more segments, against the FP64 oracle's gradient (the bounds of the
adjoint's re-traversal test: 1e-4 of the largest value, and what FP32 prefix sums allow)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2307_15333_amd import core, synth

from .test_gpu_backward import GTOL, _rel
from .test_gpu_render import oracle_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [0, 2, 3])
@pytest.mark.parametrize("cap", [4, 5, 6, 7, 8])
def test_whole_groups_and_a_part(cap, degree):
    s = synth.random_tree_scene(5, degree, seed=81 + degree, p_split=0.5)
    tree = core.Octree.from_scene(s)
    ref = oracle_tree(s)
    n = 307
    o, d = synth.random_explicit_rays(n, seed=n)
    d[1::7] *= -1.0                      # these miss the cube
    rays = core.Rays.explicit(o, d)
    g = np.random.default_rng(n).normal(size=(n, 3)).astype(np.float32)
    # a buffer that holds cap records a ray and no more
    need, more = core.Octree.records_bytes(n, cap), core.Octree.records_bytes(n, cap + 1)
    assert need < more
    rec = torch.empty(need, dtype=torch.uint8, device="cuda")
    rgb, ns, cnt = tree.render_train(rays, t_stop=0.0, records=rec)
    met = ns.cpu().numpy()
    assert (met < cap).any() and (met > cap).any()
    assert int(rec[:4].view(torch.int32)[0]) > 0
    gs = torch.zeros(tree.n_leaves, device="cuda")
    gh = torch.zeros((tree.n_leaves, 3, tree.K), device="cuda")
    tree.backward(rays, rgb, ns, torch.as_tensor(g, device="cuda"), gs, gh, t_stop=0.0, leaf_count=cnt, records=rec)
    rs, rh = O.backward(ref, o.astype(np.float64), d.astype(np.float64), g.astype(np.float64), t_stop=0.0)
    fp32 = np.sqrt(3.0) * (np.abs(g).sum(1) * (met + 4)).max() * 2.0 ** -23
    assert np.abs(gs.cpu().numpy() - rs).max() <= GTOL * np.abs(rs).max() + fp32
    assert _rel(gh.cpu().numpy(), rh) <= GTOL
