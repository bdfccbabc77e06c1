"""The order of a pixel batch inside its screen tiles: 4 x 4 cells in Morton order where the workspace has room for
their bins, tiles alone where it has only that; the content, the tiles and their order are the same."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2307_15333_amd import _lib as L
from paper_2307_15333_amd import core

from .test_zz_no_alloc import _tile_shift, _tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n_cams,n", [
    (64, 64, 100, 1 << 18),     # 2-pixel cells, many bins
    (33, 17, 3, 1600),          # few bins, ragged tiles
    (300, 200, 40, 77777),      # 8-pixel cells
    (800, 800, 100, 4096),      # sparse: tiles alone
])
@pytest.mark.parametrize("room", ["workspace()", "tiles alone"])
def test_cells_inside_tiles(W, H, n_cams, n, room):
    lib = L.load()
    ids_np = np.random.default_rng(n).choice(n_cams * W * H, n, replace=False).astype(np.int64)
    ids = torch.as_tensor(ids_np, device="cuda")
    cam, pix = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    shift = _tile_shift(n, W, H, n_cams)
    tiles = n_cams * ((W + (1 << shift) - 1) >> shift) * ((H + (1 << shift) - 1) >> shift)
    need = lib.dot_pixel_batch_workspace(n, W, H, n_cams)
    if room == "tiles alone":
        need = 4 * (2 * tiles + (tiles + 4095) // 4096 + 2 + (0 if tiles <= 4096 else n))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    L.check(lib.dot_pixel_batch(C.c_void_p(ids.data_ptr()), C.c_int64(n), W, H, n_cams, C.c_void_p(cam.data_ptr()),
                                C.c_void_p(pix.data_ptr()), C.c_void_p(out.data_ptr()), C.c_void_p(ws.data_ptr()),
                                C.c_size_t(need), core._stream()))
    cam, pix, out = cam.cpu().numpy(), pix.cpu().numpy(), out.cpu().numpy()
    assert np.array_equal(np.sort(out), np.sort(ids_np))
    assert np.array_equal(cam.astype(np.int64) * W * H + pix, out)
    t = _tiles(cam, pix, W, H, shift)
    assert np.all(np.diff(t) >= 0)
    if room == "workspace()" and n >= 8 * tiles:
        x, y = (pix % W) >> (shift - 2), (pix // W) >> (shift - 2)
        cell = (x & 1) | ((y & 1) << 1) | ((x & 2) << 1) | ((y & 2) << 2)
        assert np.all(np.diff(t * 16 + cell) >= 0)
