"""dot_build waits for its own stream alone, and several threads can build at once."""
import threading
import time

import pytest
import torch

from paper_2307_15333_amd import core, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def large():
    """2.1M leaves of degree 1: 101 MB of FP32 rows, past the size that is uploaded by several threads."""
    return synth.uniform_scene(7, 1, 0.4, seed=3)


def free_stream(streams):
    """A stream whose kernels run now: one that shares a hardware queue with a busy stream waits behind it."""
    events = []
    for s in streams:
        with torch.cuda.stream(s):
            torch.zeros(64, device="cuda").add_(1.0)
            events.append(s.record_event())
    end = time.perf_counter() + 0.3
    while time.perf_counter() < end:
        for s, e in zip(streams, events):
            if e.query():
                return s
    return None


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_build_beside_a_busy_stream(large, storage):
    sigma, sh = large.sigma, large.sh
    streams = [torch.cuda.Stream() for _ in range(6)]
    for s in streams:                            # blocks of the planes' sizes for the allocator to reuse
        with torch.cuda.stream(s):
            core.Octree(large.child, sigma, sh, 1, storage).close()
    busy = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(int(2.4e9))            # about a second
        done = busy.record_event()
    s = free_stream(streams)
    assert s is not None
    with torch.cuda.stream(s):
        tree = core.Octree(large.child, sigma, sh, 1, storage)
    assert not done.query()                      # the build did not wait for it
    busy.synchronize()
    dt = {"f32": torch.float32, "f16": torch.float16}[storage]
    assert torch.equal(tree.plane_views()[1].cpu(), torch.from_numpy(sh).to(dt))


def test_builds_from_two_threads(large):
    """One of them finds the pinned slots in use and copies by itself."""
    trees, errors = [None, None], []

    def build(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                trees[k] = core.Octree.from_scene(large)
        except Exception as e:      # reported by the test's thread
            errors.append(e)

    ts = [threading.Thread(target=build, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    for t in trees:
        assert torch.equal(t.plane_views()[1].cpu(), torch.from_numpy(large.sh))
