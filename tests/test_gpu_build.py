"""Uploading planes large enough to be copied by several host threads: every value arrives where it belongs, stored as
it is (FP32 rows without padding), padded (degree 2) or rounded to 16 bits."""
import numpy as np
import pytest
import torch

from paper_2307_15333_amd import core, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,degree", [("f32", 1), ("f32", 2), ("f16", 1), ("bf16", 2)])
def test_threaded_upload(storage, degree):
    s = synth.uniform_scene(7, degree, 5.0, seed=degree)     # 2^21 leaves: 100 or 226 MB, the last chunk partial
    tree = core.Octree.from_scene(s, storage)
    sigma, sh = tree.plane_views()
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    assert torch.equal(sh.cpu(), torch.from_numpy(s.sh32).to(dt))
    assert torch.equal(sigma.cpu(), torch.from_numpy(s.sigma).to(dt))
    if storage == "f32" and degree == 2:
        i = tree.info()
        rows = tree.alloc.tensor(i.sh, s.n_leaves * i.sh_stride * 4).view(torch.float32).view(s.n_leaves, -1)
        assert (rows[:, 27:] == 0).all()
