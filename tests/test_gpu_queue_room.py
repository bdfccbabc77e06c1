"""An open serving queue leaves room for other work: kernels of other streams run and trees are built beside it, in
every storage type of the queue, and it renders trees without links too."""
import time

import numpy as np
import pytest
import torch

from paper_2307_15333_amd import core, serve, synth

pytestmark = pytest.mark.gpu

CAM = synth.look_at_camera(20.0, 10.0, 4.0, 64, 48)


def small_tree(storage, degree=3):
    tree = core.Octree.from_scene(synth.random_tree_scene(5, degree, seed=2, p_split=0.5),
                                  "f16" if storage == "pal16" else storage)
    if storage == "pal16":
        tree.quantize_sh(6)
    return tree


def streams_that_run(streams, work, seconds):
    """Those of the streams whose work completes in time (one that shares a hardware queue with the launch waits)."""
    events = []
    for s, f in zip(streams, work):
        with torch.cuda.stream(s):
            f()
            events.append(s.record_event())
    end = time.perf_counter() + seconds
    while time.perf_counter() < end and not all(e.query() for e in events):
        time.sleep(0.001)
    return [s for s, e in zip(streams, events) if e.query()]


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16", "pal16"])
@pytest.mark.parametrize("work", ["fill", "render", "train"])
def test_other_kernels_run_beside_an_open_queue(storage, work):
    """A small kernel, and the library's own of about 128 and 144 registers a lane."""
    tree = small_tree(storage)
    want = tree.render(core.Rays.cameras(np.asarray(CAM).reshape(1))).reshape(48, 64, 3)
    outs = [torch.zeros((48, 64, 3), device="cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(5)]
    buffers = [torch.zeros(1 << 20, device="cuda") for _ in streams]
    other = small_tree("f32")
    rays = core.Rays.cameras(synth.random_sphere_cameras(2, 4.0, 100, 80, 1))
    fs = {"fill": [lambda b=b: b.add_(1.0) for b in buffers], "render": [lambda: other.render(rays)] * 5,
          "train": [lambda: other.render_train(rays)] * 5}[work]
    for s, f in zip(streams, fs):
        with torch.cuda.stream(s):
            f()
    torch.cuda.synchronize()
    q = serve.Queue(storage, max_jobs=8, max_seconds=3.0)
    try:
        q.wait(q.push(tree, CAM, outs[0], 64, 48))
        ran = streams_that_run(streams, fs, 0.3)
        q.wait(q.push(tree, CAM, outs[1], 64, 48))      # it is still open
    finally:
        q.close()
    assert len(ran) >= 2
    assert torch.equal(outs[0], want) and torch.equal(outs[1], want)


def test_build_beside_an_open_queue():
    """101 MB of rows (uploaded by several threads) and the links' kernels."""
    large = synth.uniform_scene(7, 1, 0.4, seed=3)
    sigma, sh = large.sigma, large.sh
    tree = small_tree("f16")
    out = torch.zeros((48, 64, 3), device="cuda")
    streams = [torch.cuda.Stream() for _ in range(5)]
    buffers = [torch.zeros(64, device="cuda") for _ in streams]
    for s, b in zip(streams, buffers):                   # blocks of the planes' sizes for the allocator to reuse
        with torch.cuda.stream(s):
            b.add_(1.0)
            core.Octree(large.child, sigma, sh, 1).close()
    torch.cuda.synchronize()
    q = serve.Queue("f16", max_jobs=8, max_seconds=6.0)
    try:
        q.wait(q.push(tree, CAM, out, 64, 48))
        ran = streams_that_run(streams, [lambda b=b: b.add_(1.0) for b in buffers], 0.3)
        assert ran
        with torch.cuda.stream(ran[0]):
            built = core.Octree(large.child, sigma, sh, 1)
        q.wait(q.push(tree, CAM, out, 64, 48))           # the launch has not ended: the build did not wait for it
    finally:
        q.close()
    assert torch.equal(built.plane_views()[1].cpu(), torch.from_numpy(sh))


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_queue_renders_trees_without_links(storage):
    trees = [small_tree(storage, 3), small_tree(storage, 1)]
    trees[0].set_links(False)
    rays = core.Rays.cameras(np.asarray(CAM).reshape(1))
    want = [t.render(rays).reshape(48, 64, 3) for t in trees]
    outs = [torch.zeros((48, 64, 3), device="cuda") for _ in trees]
    torch.cuda.synchronize()
    q = serve.Queue(storage, max_jobs=8, max_seconds=5.0)
    try:
        for tk in [q.push(t, CAM, o, 64, 48) for t, o in zip(trees, outs)]:
            q.wait(tk)
    finally:
        q.close()
    for o, w in zip(outs, want):
        assert torch.equal(o, w)
