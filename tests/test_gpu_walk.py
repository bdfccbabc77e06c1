"""The forward walk's edges on the GPU: lanes without a ray beside lanes with one, rays along the axes and in cell
planes, trees past the reach of 32-bit plane offsets, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2307_15333_amd import core, synth

from .test_gpu_render import TOL32, oracle_tree, rgb_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("storage,degree", [("f32", 3), ("f32", 2), ("f32", 0), ("f16", 3), ("bf16", 1)])
def test_partial_quads_and_waves(storage, degree, links):
    """Ray counts that leave lanes of a quad or waves of a workgroup empty; half of the rays miss the cube."""
    s = synth.random_tree_scene(5, degree, seed=31 + degree, p_split=0.5)
    tree = core.Octree.from_scene(s, storage)
    tree.set_links(links)
    ref_tree = oracle_tree(s, storage)
    for n in (1, 2, 3, 5, 63, 65, 130):
        o, d = synth.random_explicit_rays(n, seed=n)
        d[1::2] *= -1.0
        rgb, ns = tree.render(core.Rays.explicit(o, d), nseg=True)
        ref = O.render(ref_tree, o, d)
        assert rgb_err(rgb.cpu().numpy(), ref).max() <= TOL32
        assert (ns.cpu().numpy()[1::2] == 0).all()


@pytest.mark.parametrize("links", [True, False])
def test_axis_rays_and_cell_planes(links):
    """Directions with zero (and negative zero) components, in cell planes and on the cube's faces and edges."""
    s = synth.random_tree_scene(4, 3, seed=5, p_split=0.6)
    tree = core.Octree.from_scene(s)
    tree.set_links(links)
    at = np.array([-1.0, -0.75, -0.3, 0.0, 0.5, 0.7, 1.0])
    o, d = [], []
    for a in range(3):
        for sgn in (1.0, -1.0):
            for u in at:
                for v in at:
                    p = np.insert([u, v], a, -2.0 * sgn)
                    q = np.full(3, -0.0)
                    q[a] = sgn
                    o.append(p)
                    d.append(q)
    # diagonals: several axes attain the exit at once
    for sx in (1.0, -1.0):
        for sy in (1.0, -1.0):
            o.append([-2.0 * sx, -2.0 * sy, 0.25])
            d.append([sx, sy, 0.0])
            o.append([-2.0 * sx, -2.0 * sy, -2.0])
            d.append([sx, sy, 1.0])
    o, d = np.array(o, np.float32), np.array(d, np.float32)
    rgb = tree.render(core.Rays.explicit(o, d), t_stop=0.0)
    ref = O.render(O.OracleTree.from_scene(s, sigma=s.sigma.astype(np.float64)), o, d, t_stop=0.0)
    assert np.abs(rgb.cpu().numpy() - ref["rgb"]).max() <= TOL32


def test_tree_past_32bit_offsets():
    """28.5M FP32 leaves of degree 3 (5.5 GB of rows), grown by refinement from 2.1M: subdividing a leaf does not
    change the image, so it is the small tree's.  A ray crosses at most 3 * 2^9 + 64 leaves; each addition to the
    optical depth S rounds by 2^-24 S and moves the colour by at most T S 2^-24 <= 2^-24 / e, each weighted colour
    by 2^-24: 1600 * 2^-24 * (1 + 1/e) = 1.3e-4."""
    s = synth.uniform_scene(7, 3, 0.4, seed=3)
    tree = core.Octree.from_scene(s)
    rays = core.Rays.cameras(synth.cameras([(30.0, 20.0, 4.0, 61, 45)]))
    small = tree.render(rays, t_stop=0.0).cpu().numpy()
    assert tree.info().sh_stride * 4 * tree.n_leaves < 2 ** 32
    for frac in (1.0, 0.1):
        tree.refine(torch.rand(tree.n_leaves, device="cuda") + 0.5, prune_tau=0.0, sample_frac=frac, max_depth=12)
    assert tree.info().sh_stride * 4 * tree.n_leaves > 2 ** 32
    for links in (True, False):
        tree.set_links(links)
        assert np.abs(tree.render(rays, t_stop=0.0).cpu().numpy() - small).max() <= 1.3e-4


@pytest.mark.parametrize("views,w,h", [(1, 128, 63), (1, 128, 64), (1, 136, 72), (3, 77, 51), (8, 40, 33), (9, 64, 48)])
def test_bands_cover_every_pixel(views, w, h):
    """Whole views are handed to the XCDs in bands (63 to 65 workgroups: none, one tile row or a remainder); the same
    pixels given as a list take another order."""
    s = synth.random_tree_scene(4, 1, seed=9, p_split=0.5)
    tree = core.Octree.from_scene(s)
    cams = synth.random_sphere_cameras(views, 3.5, w, h, seed=views)
    rgb = tree.render(core.Rays.cameras(cams))
    i = np.arange(views * w * h)
    listed = tree.render(core.Rays.pixels(cams, i // (w * h), i % (w * h)))
    assert torch.equal(rgb, listed)


@pytest.mark.parametrize("storage,degree", [("f32", 3), ("f32", 0), ("f16", 2), ("bf16", 3)])
@pytest.mark.parametrize("mode", ["max", "sum"])
def test_signal_alone_equals_fused_signal(storage, degree, mode):
    """The signal pass fetches no rows; its weights are the fused render's (the sum's order may differ)."""
    s = synth.random_tree_scene(5, degree, seed=17, p_split=0.5)
    tree = core.Octree.from_scene(s, storage)
    rays = core.Rays.cameras(synth.random_sphere_cameras(3, 3.5, 45, 31, seed=2))
    fused, alone = (torch.full((tree.n_leaves,), 0.25, device="cuda") for _ in range(2))
    tree.render(rays, signal=fused, signal_mode=mode)
    tree.accumulate_signal(rays, alone, signal_mode=mode)
    if mode == "max":
        assert torch.equal(fused, alone)
    else:       # n additions of weights in [0, 1] in another order: n 2^-24 of the sum, n <= 4185 rays
        torch.testing.assert_close(fused, alone, rtol=4185 * 2.0 ** -24, atol=0)


@pytest.mark.parametrize("links", [(True, True), (True, False)])
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_jobs_batch_equals_render(storage, links):
    """A batch of jobs, down to a single tile, over trees that all have links and over a mix (another kernel)."""
    from paper_2307_15333_amd import serve
    trees = []
    for k, on in enumerate(links):
        t = core.Octree.from_scene(synth.random_tree_scene(5, 3 - k, seed=40 + k, p_split=0.5), storage)
        t.set_links(on)
        trees.append(t)
    for sizes in ([(7, 5)], [(64, 40), (9, 200), (33, 31), (128, 8)]):
        reqs = [serve.Request(rid=i, tree=i % 2, cam=synth.cameras([(40.0 * i, 10.0, 4.0, w, h)])[0], width=w, height=h,
                              arrival=0.0) for i, (w, h) in enumerate(sizes)]
        serve.Server(trees).run(reqs, keep_outputs=True)
        for r in reqs:
            want = trees[r.tree].render(core.Rays.cameras(np.array([r.cam])))
            assert torch.equal(r.out.reshape(-1, 3), want)
