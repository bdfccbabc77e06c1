"""The order of a pixel batch does not depend on how much larger than asked for its workspace is (one that is kept from
another call), up to and past the batches whose cells are ordered."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2307_15333_amd import _lib as L
from paper_2307_15333_amd import core

from .test_zz_no_alloc import _tile_shift, _tiles

pytestmark = pytest.mark.gpu


def _cells_ordered(cam, pix, W, H, shift):
    t = _tiles(cam, pix, W, H, shift)
    assert np.all(np.diff(t) >= 0)
    x, y = (pix % W) >> (shift - 2), (pix // W) >> (shift - 2)
    return bool(np.all(np.diff(t * 16 + ((x & 1) | ((y & 1) << 1) | ((x & 2) << 1) | ((y & 2) << 2))) >= 0))


@pytest.mark.parametrize("W,H,n_cams,n,cells", [(64, 64, 100, 4000, True), (800, 800, 100, 1 << 20, True),
                                                (800, 800, 100, 3 << 20, False), (800, 800, 100, 1 << 16, False)])
def test_a_larger_workspace_gives_the_same_order(W, H, n_cams, n, cells):
    lib = L.load()
    ids = torch.randperm(n_cams * W * H, device="cuda", generator=torch.Generator("cuda").manual_seed(1))[:n].contiguous()
    shift = _tile_shift(n, W, H, n_cams)
    need = lib.dot_pixel_batch_workspace(n, W, H, n_cams)
    for room in (need, 8 * need + (64 << 20)):
        cam, pix = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
        ws = torch.empty(room, dtype=torch.uint8, device="cuda")
        L.check(lib.dot_pixel_batch(C.c_void_p(ids.data_ptr()), C.c_int64(n), W, H, n_cams, C.c_void_p(cam.data_ptr()),
                                    C.c_void_p(pix.data_ptr()), None, C.c_void_p(ws.data_ptr()), C.c_size_t(room),
                                    core._stream()))
        flat = cam.long() * (W * H) + pix
        assert torch.equal(flat.sort()[0], ids.sort()[0])
        assert _cells_ordered(cam.cpu().numpy(), pix.cpu().numpy(), W, H, shift) == cells
