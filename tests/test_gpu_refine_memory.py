"""The device memory that a refinement holds at its peak: the two trees' planes, 48 bytes of scratch a leaf, a row and
36 bytes an internal node, whether no leaves are subdivided or half of them."""
import pytest
import torch

from paper_2307_15333_amd import core, synth

pytestmark = pytest.mark.gpu


class CountingAllocator(core.TorchAllocator):
    def __init__(self, device):
        self.live = self.peak = 0
        super().__init__(device)

    def _alloc(self, nbytes, ctx):
        p = super()._alloc(nbytes, ctx)
        if p is not None:
            self.live += int(nbytes)
            self.peak = max(self.peak, self.live)
        return p

    def _free(self, p, ctx):
        if p in self.blocks:
            self.live -= self.blocks[p].numel()
        super()._free(p, ctx)


def _planes(leaves, internal, row):
    return leaves * (4 + row + 1) + internal * 32


@pytest.mark.parametrize("frac", [0.0, 0.05, 0.5])
def test_peak_of_a_refinement(frac, monkeypatch):
    monkeypatch.setattr(core, "TorchAllocator", CountingAllocator)
    s = synth.make_scene(synth.sdf_sphere(0.5), max_depth=6, degree=3, seed=1)
    tree = core.Octree.from_scene(s)
    L, I, row = tree.n_leaves, tree.n_internal, 192
    gen = torch.Generator("cuda").manual_seed(1)
    sig = torch.rand(L, device="cuda", generator=gen)
    tree.alloc.peak = tree.alloc.live
    st = tree.refine(sig, prune_tau=0.0, sample_frac=frac, max_depth=12)
    L2, I2 = st["leaves_after"], st["internal_after"]
    # the old links stay until the new tree is complete
    assert tree.alloc.peak <= _planes(L, I, row) + 24 * L + _planes(L2, I2, row) + 48 * L + I * (32 + row + 4) + (1 << 16)
    tree.close()
