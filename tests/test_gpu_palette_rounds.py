"""The median cut's two kinds of round (boxes shared by workgroups, boxes of one workgroup) at the sizes where they
change over, with ties, signed zeros and constant dimensions, against the oracle: indices and palette are the same."""
import dataclasses

import numpy as np
import pytest

from paper_2307_15333_amd import synth

from .test_gpu_palette import _f16_ulps, _quantize_both

pytestmark = pytest.mark.gpu


def _rows(n, degree, kind, seed):
    rng = np.random.default_rng(seed)
    K = (degree + 1) ** 2
    x = rng.standard_normal((n, 3, K)).astype(np.float32)
    if kind == "ties":          # a few values, signed zeros among them
        x = np.round(x).astype(np.float32) * np.float32(0.5)
        x[rng.random(x.shape) < 0.3] = -0.0
    elif kind == "flat":        # one dimension varies, by the last bits of its value
        x[:] = 0.25
        x[:, 1, K - 1] = (0x3f800000 + rng.integers(0, 64, n)).astype(np.uint32).view(np.float32)
    return x


@pytest.mark.parametrize("storage,degree,kind,bits", [
    ("f32", 3, "normal", 6), ("f32", 1, "ties", 5), ("f32", 0, "flat", 4), ("f32", 2, "flat", 9), ("f16", 2, "ties", 7),
    ("bf16", 3, "normal", 3)])
@pytest.mark.parametrize("depth", [3, 4, 5])
def test_rounds_match_oracle(storage, degree, kind, bits, depth):
    """512, 4096 and 32768 leaves: boxes of 32768 down to 1 member, 4096 and 1024 being the changes of kernel."""
    s = synth.uniform_scene(depth, degree, 1.0)
    s = dataclasses.replace(s, sh32=_rows(s.n_leaves, degree, kind, depth))
    tree, _, idx, pal, (_, want_idx, want_pal, _) = _quantize_both(s, bits, storage)
    tree.close()
    assert np.array_equal(idx, want_idx)
    assert _f16_ulps(pal, want_pal).max() <= 1
