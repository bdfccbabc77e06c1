"""The adjoint's own walks of the tree (without records, and past a ray's record capacity) against the FP64 oracle's
gradient: every storage type, with and without links, ray counts that leave lanes and waves empty.

The tolerance is the gradients' usual 1e-4 of the largest value plus what FP32 prefix sums allow: a segment's
dL/dsigma = delta sum_ch g_ch (T c - (C - P)) takes the difference of two sums of N colours that add up to at most 1,
each rounded N times (2^-24 a time), and delta <= sqrt(3) (cells of edge 1 at most), so a ray of N segments may be
off by sqrt(3) |g|_1 (N + 4) 2^-23 where nothing cancels."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2307_15333_amd import core, synth

from .test_gpu_backward import GTOL, _rel
from .test_gpu_render import oracle_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("storage,degree,records", [("f32", 3, None), ("f32", 3, 3), ("f32", 2, 3), ("f32", 1, 1), ("f32", 0, 3),
                                                    ("f16", 3, None), ("bf16", 1, None), ("f16", 0, None)])
def test_walks_of_the_adjoint(storage, degree, records, links):
    s = synth.random_tree_scene(5, degree, seed=81 + degree, p_split=0.5)
    tree = core.Octree.from_scene(s, storage)
    tree.set_links(links)
    ref = oracle_tree(s, storage)
    for n in (1, 67, 500):
        o, d = synth.random_explicit_rays(n, seed=n)
        d[1::3] *= -1.0                      # these miss the cube
        rays = core.Rays.explicit(o, d)
        g = np.random.default_rng(n).normal(size=(n, 3)).astype(np.float32)
        g[::5] = 0.0 if n > 1 else g[::5]    # and these have no gradient
        cnt = rec = None
        if records is None:
            rgb, ns = tree.render(rays, t_stop=0.0, nseg=True)
        else:
            rec = torch.empty(core.Octree.records_bytes(n, records), dtype=torch.uint8, device="cuda")
            rgb, ns, cnt = tree.render_train(rays, t_stop=0.0, records=rec)
        gs = torch.zeros(tree.n_leaves, device="cuda")
        gh = torch.zeros((tree.n_leaves, 3, tree.K), device="cuda")
        tree.backward(rays, rgb, ns, torch.as_tensor(g, device="cuda"), gs, gh, t_stop=0.0, leaf_count=cnt, records=rec)
        rs, rh = O.backward(ref, o.astype(np.float64), d.astype(np.float64), g.astype(np.float64), t_stop=0.0)
        fp32 = np.sqrt(3.0) * (np.abs(g).sum(1) * (ns.cpu().numpy() + 4)).max() * 2.0 ** -23
        assert np.abs(gs.cpu().numpy() - rs).max() <= GTOL * np.abs(rs).max() + fp32
        assert _rel(gh.cpu().numpy(), rh) <= GTOL
    tree.close()
