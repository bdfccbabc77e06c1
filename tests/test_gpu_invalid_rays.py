"""Rays without a valid direction or origin (an all-zero direction, a broken camera) beside ordinary ones: they end at
once, visibly (a NaN colour from their first leaf; nothing composited where only the origin is not a number), and the
rays beside them are untouched."""
import numpy as np
import pytest
import torch

from paper_2307_15333_amd import core, serve, synth

pytestmark = pytest.mark.gpu

NAN, INF = np.nan, np.inf
BAD = np.array([[0, 0, 0], [NAN, NAN, NAN], [NAN, 0, 0], [0, 1, NAN], [INF, 0, 0], [-INF, INF, 0]], np.float32)


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("storage,degree", [("f32", 3), ("f32", 1), ("f16", 3), ("bf16", 2)])
def test_rays_without_a_direction(storage, degree, links):
    s = synth.random_tree_scene(6, degree, seed=61 + degree, p_split=0.5)
    tree = core.Octree.from_scene(s, storage)
    tree.set_links(links)
    o, d = synth.random_explicit_rays(131, seed=4)
    calls = [lambda r: tree.render(r, nseg=True)]
    if storage == "f32":
        calls.append(lambda r: tree.render_train(r)[:2])
    bad = np.arange(1, 131, 5)
    o2, d2 = o.copy(), d.copy()
    d2[bad] = BAD[np.arange(bad.size) % len(BAD)]
    o2[bad] = 0.25
    rays = core.Rays.explicit(o2, d2)
    good = np.setdiff1d(np.arange(131), bad)
    for call in calls:
        want, want_ns = call(core.Rays.explicit(o, d))
        rgb, ns = call(rays)
        assert torch.equal(rgb[good], want[good]) and torch.equal(ns[good], want_ns[good])
        assert torch.isnan(rgb[bad]).all()
        assert (ns[bad] == 1).all()
    # found from the root once, and no further
    st = tree.render_stats(core.Rays.explicit(o2[bad], d2[bad]))
    assert st["segments"] == bad.size and st["index_reads"] <= bad.size * int(tree.info().max_depth)


@pytest.mark.parametrize("links", [True, False])
def test_origin_that_is_not_a_number(links):
    tree = core.Octree.from_scene(synth.random_tree_scene(6, 3, seed=7, p_split=0.5))
    tree.set_links(links)
    o = np.full((3, 3), NAN, np.float32)
    d = np.array([[1, 0, 0], [0.6, 0.8, 0], [-0.6, 0.48, 0.64]], np.float32)
    rays = core.Rays.explicit(o[2:], d[2:])
    rgb, ns = tree.render(rays, bg=(0.25, 0.5, 0.75), nseg=True)
    assert torch.equal(rgb.cpu(), torch.tensor([[0.25, 0.5, 0.75]])) and int(ns[0]) == 0


def test_camera_without_a_focal_length():
    """Views and served requests."""
    tree = core.Octree.from_scene(synth.random_tree_scene(6, 3, seed=8, p_split=0.5), "f16")
    cams = synth.cameras([(30.0, 20.0, 4.0, 40, 24), (80.0, -10.0, 4.0, 40, 24)])
    want = tree.render(core.Rays.cameras(cams)).reshape(2, 24, 40, 3)
    cams["c2w"][1] = NAN
    rgb = tree.render(core.Rays.cameras(cams)).reshape(2, 24, 40, 3)
    assert torch.equal(rgb[0], want[0])
    assert torch.isnan(rgb[1]).all()
    reqs = [serve.Request(rid=i, tree=0, cam=cams[i], width=40, height=24, arrival=0.0) for i in range(2)]
    serve.Server([tree]).run(reqs, keep_outputs=True)
    assert torch.equal(reqs[0].out, want[0])
    assert torch.isnan(reqs[1].out).all()
