"""Refinement's row kernels at the widths they can go wrong: one piece a row (degree 0), rows whose last piece is part
padding (degree 2), 16-bit rows, trees of fewer rows than a workgroup takes; and the refined tree's depth."""
import numpy as np
import pytest
import torch

from paper_2307_15333_amd import core, synth

from .test_gpu_refine import _compare, _seeded_signal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("recursive,reinit", [(False, False), (True, False), (False, True)])
def test_rows_of_every_width(degree, storage, recursive, reinit):
    s = synth.random_tree_scene(4, degree, seed=60 + degree, p_split=0.55)
    st, _ = _compare(s, _seeded_signal(s.n_leaves, degree, 0.92), storage, prune_tau=2e-3, sample_frac=0.05, max_depth=6,
                     recursive=recursive, reinit=reinit)
    assert st["merged"] > 0 and st["subdivided"] > 0


@pytest.mark.parametrize("frac,tau", [(0.0, 0.0), (1.0, 0.0), (0.0, 2.0), (0.02, 0.5)])
def test_depth_of_the_refined_tree(frac, tau):
    s = synth.random_tree_scene(3, 1, seed=4, p_split=0.4)
    tree = core.Octree.from_scene(s)
    for k in range(3):
        sig = torch.as_tensor(np.random.default_rng(k).uniform(0.01, 1.0, tree.n_leaves).astype(np.float32), device="cuda")
        tree.refine(sig, prune_tau=tau, sample_frac=frac, max_depth=8)
        assert tree.info().max_depth == int(tree.export()["depth"].max())
