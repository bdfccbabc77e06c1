"""Trees with a plane past the reach of 32-bit offsets (28.5M FP32 leaves of degree 3: 5.5 GB of rows), which every path
walks lane by lane: training forward, adjoint with records, past their capacity and without them, signals, served
batches and the persistent queue.

The tree is grown by refinement from a uniform one of 2.1M leaves.  Subdividing a leaf changes no image, so a leaf's
gradient, and its summed signal, is the sum over the leaves it became; the small tree's come from the wave-wide walk.
N <= 3 * 2^9 + 64 segments of a ray: an addition to the optical depth rounds by 2^-24 S, so T is off by N 2^-24 / e and a
weight by twice that and a rounding (7.2e-5); a leaf met by m rays takes m of those."""
import numpy as np
import pytest
import torch

from paper_2307_15333_amd import core, serve, synth

from .test_gpu_backward import GTOL

pytestmark = pytest.mark.gpu

N_SEG = 3 * 2 ** 9 + 64
W_ERR = 2 * N_SEG * 2.0 ** -24 / np.e + 16 * 2.0 ** -24


@pytest.fixture(scope="module")
def trees():
    s = synth.uniform_scene(7, 3, 0.4, seed=3)
    small, far = core.Octree.from_scene(s), core.Octree.from_scene(s)
    gen = torch.Generator("cuda").manual_seed(1)
    for frac in (1.0, 0.1):
        far.refine(torch.rand(far.n_leaves, device="cuda", generator=gen) + 0.5, prune_tau=0.0, sample_frac=frac, max_depth=12)
    info = far.info()
    assert info.sh_stride * 4 * far.n_leaves > 2 ** 32 and info.max_depth == 9
    # the small tree's leaf that each leaf was: leaves lie in Morton order, a leaf of depth d holds 8^(9 - d) finest cells
    depth = far.alloc.tensor(info.leaf_depth, far.n_leaves)
    cells = torch.pow(8, 9 - depth.long())
    parent = (cells.cumsum(0) - cells) // 64
    assert int(parent[-1]) == small.n_leaves - 1
    yield small, far, parent
    small.close()
    far.close()


def _summed(x, parent, n):
    return torch.zeros((n, *x.shape[1:]), device="cuda", dtype=torch.float64).index_add_(0, parent, x.double())


@pytest.fixture(scope="module")
def small_adjoint(trees):
    small = trees[0]
    rays = core.Rays.cameras(synth.cameras([(30.0, 20.0, 4.0, 61, 45)]))
    g = torch.randn((rays.n_rays, 3), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    rgb, ns, cnt = small.render_train(rays, t_stop=0.0)
    gs = torch.zeros(small.n_leaves, device="cuda")
    gh = torch.zeros((small.n_leaves, 3, 16), device="cuda")
    small.backward(rays, rgb, ns, g, gs, gh, t_stop=0.0, leaf_count=cnt)
    return rays, g, rgb, gs, gh, int(cnt.sum(0).max())


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("records", [None, 5, 24, 640, "counts only"])
def test_far_training(trees, small_adjoint, records, links):
    small, far, parent = trees
    rays, g, want, gs0, gh0, m = small_adjoint
    far.set_links(links)
    cnt = rec = None
    if records is None:
        rgb, ns = far.render(rays, t_stop=0.0, nseg=True)
    else:
        if records != "counts only":
            rec = torch.empty(core.Octree.records_bytes(rays.n_rays, records), dtype=torch.uint8, device="cuda")
        rgb, ns, cnt = far.render_train(rays, t_stop=0.0, records=rec)
        if records == 24:
            assert 0 < int(rec[:4].view(torch.int32)[0]) < rays.n_rays      # some rays overflow
    assert (rgb - want).abs().max() <= 1.3e-4        # the bound of the plain render's test
    gs = torch.zeros(far.n_leaves, device="cuda")
    gh = torch.zeros((far.n_leaves, 3, 16), device="cuda")
    far.backward(rays, rgb, ns, g, gs, gh, t_stop=0.0, leaf_count=cnt, records=rec)
    g1 = float(g.abs().sum(1).max())
    edge = np.sqrt(3.0) * 2.0 / 128
    assert (_summed(gs, parent, small.n_leaves) - gs0).abs().max() <= GTOL * float(gs0.abs().max()) + 2 * m * edge * g1 * (N_SEG + 4) * 2.0 ** -23
    assert (_summed(gh, parent, small.n_leaves) - gh0).abs().max() <= GTOL * float(gh0.abs().max()) + m * g1 * W_ERR * 0.25 * 1.1


def test_far_fused_step_equals_the_separate_one(trees, small_adjoint):
    """The optimiser inside the adjoint reads and writes the same planes past 4 GiB (lr 0: the planes stay)."""
    _, far, _ = trees
    rays, g, *_ = small_adjoint
    far.set_links(True)
    rec = torch.empty(core.Octree.records_bytes(rays.n_rays, 24), dtype=torch.uint8, device="cuda")
    rgb, ns, cnt = far.render_train(rays, t_stop=0.0, records=rec)
    kw = dict(t_stop=0.0, leaf_count=cnt, records=rec)
    gs = torch.zeros(far.n_leaves, device="cuda")
    gh = torch.zeros((far.n_leaves, 3, 16), device="cuda")
    far.backward(rays, rgb, ns, g, gs, gh, **kw)
    st = far.rmsprop_state()
    far.backward_rmsprop(rays, rgb, ns, g, st, lr_sigma=0.0, lr_sh=0.0, alpha=0.0, **kw)
    # the square averages are the squared gradients (rows past a ray's records take their slots in any order)
    torch.testing.assert_close(st["v_sigma"].sqrt(), gs.abs(), rtol=1e-4, atol=1e-4 * float(gs.abs().max()))
    torch.testing.assert_close(st["v_sh"].sqrt(), gh.abs(), rtol=1e-4, atol=1e-4 * float(gh.abs().max()))


def test_far_signals(trees, small_adjoint):
    small, far, parent = trees
    rays, m = small_adjoint[0], small_adjoint[5]
    far.set_links(True)
    want = torch.zeros(small.n_leaves, device="cuda")
    small.accumulate_signal(rays, want, t_stop=0.0, signal_mode="sum")
    outs = [torch.zeros(far.n_leaves, device="cuda") for _ in range(3)]
    far.accumulate_signal(rays, outs[0], t_stop=0.0, signal_mode="sum")
    far.render(rays, t_stop=0.0, signal=outs[1], signal_mode="sum")
    far.render_train(rays, t_stop=0.0, signal=outs[2], signal_mode="sum")
    for out in outs:
        assert (_summed(out, parent, small.n_leaves) - want).abs().max() <= m * W_ERR
    # one ray: the largest weight of a leaf is the sum of its weights
    one = core.Rays.explicit([[-3.0, 0.1, 0.2]], [[1.0, 0.02, -0.03]])
    a, b, c = (torch.zeros(far.n_leaves, device="cuda") for _ in range(3))
    far.accumulate_signal(one, a, t_stop=0.0, signal_mode="sum")
    far.accumulate_signal(one, b, t_stop=0.0)
    far.render(one, t_stop=0.0, signal=c)
    assert int((a > 0).sum()) > 100 and torch.equal(a, b) and torch.equal(a, c)


def test_far_tree_is_served(trees):
    """Beside a tree with 32-bit offsets, in a batch of jobs and in the persistent queue."""
    small, far, _ = trees
    for links in (True, False):
        far.set_links(links)
        cams = [synth.look_at_camera(20.0 + 50 * i, 10.0, 4.0, 72, 41) for i in range(3)]
        want = [t.render(core.Rays.cameras(np.asarray(c).reshape(1))).reshape(41, 72, 3)
                for t, c in zip((far, small, far), cams)]
        reqs = [serve.Request(rid=i, tree=i % 2, cam=cams[i], width=72, height=41, arrival=0.0) for i in range(3)]
        serve.Server([far, small]).run(reqs, keep_outputs=True)
        outs = [torch.zeros((41, 72, 3), device="cuda") for _ in range(3)]
        torch.cuda.synchronize()
        q = serve.Queue("f32", max_jobs=8, max_seconds=10.0)
        try:
            for tk in [q.push(t, c, o, 72, 41) for t, c, o in zip((far, small, far), cams, outs)]:
                q.wait(tk)
        finally:
            q.close()
        for r, o, w in zip(reqs, outs, want):
            assert torch.equal(r.out, w) and torch.equal(o, w)
