"""GPU: device memory that solves take through the allocation callback beside their vectors - the assembled
stencils of the coarse levels."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gmt_inputs import gyroid_sheet, uniform  # noqa: E402
from paper_2604_26518_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda"


class Recorder(B._TorchArena):
    """The default arena, with the sizes of the allocations made."""

    def __init__(self, device):
        self.made = []
        self.size = {}
        super().__init__(device)

    def _alloc(self, nbytes, ctx):
        ptr = super()._alloc(nbytes, ctx)
        if ptr is not None:
            self.made.append(int(nbytes))
            self.size[ptr] = int(nbytes)
        return ptr

    def _release(self, ptr, ctx):
        self.size.pop(ptr, None)
        super()._release(ptr, ctx)


def _load(H):
    """A load that is not zero on the full cell either."""
    g = torch.Generator(device=DEV).manual_seed(1)
    return H.apply_K(torch.randn((H.n_n(), H.c, H.d), generator=g, device=DEV, dtype=torch.float64))


def _stencil_bytes(H, l):
    return H.n_n(l) * 28 * H.d ** 2 * 4 + 16  # FP32: 27 blocks and one of padding; the library adds 16


@pytest.mark.parametrize("N,L,phys", [(24, 3, "thermal"), (48, 4, "thermal"), (64, 5, "thermal"), (32, 4, "elastic")])
@pytest.mark.parametrize("family", ["gyroid", "uniform"])
def test_stencils_are_held_where_a_sweep_takes_them(family, N, L, phys, monkeypatch):
    """A level whose solves take the element matrices holds no stencils afterwards, and the next hierarchy
    of the class, whose choice is known, lays out exactly those that the first one kept."""
    monkeypatch.setattr(B, "_TorchArena", Recorder)
    vox = gyroid_sheet(N, 0, 0.3) if family == "gyroid" else uniform(N)
    kept = []
    for turn in range(2):
        H = B.Hierarchy(vox, L, phys)
        f = _load(H)
        before = len(H._arena.made)
        H.solve(f, precision="f32", tol=1e-3)
        made = H._arena.made[before:]
        live = list(H._arena.size.values())
        kept.append([l for l in range(2, L) if live.count(_stencil_bytes(H, l)) > 0])
        if turn == 1:
            assert kept[1] == kept[0]
            assert [l for l in range(2, L) if _stencil_bytes(H, l) in made] == kept[0]
        H.close()
    print(f"[{family} {N} {phys}] stencils kept on levels {kept[0]} of 2..{L - 1}", flush=True)


@pytest.mark.parametrize("density", [False, True])
def test_no_stencils_where_no_sweep_takes_them(density, monkeypatch):
    """With the coarse sweeps pinned to the element matrices a solve lays no stencils out."""
    monkeypatch.setattr(B, "_TorchArena", Recorder)
    monkeypatch.setenv("GMT_FORCE_COARSE_VARIANT", "1")
    vox = gyroid_sheet(32, 0, 0.3)
    H = B.Hierarchy(None, 4, "elastic", density=0.5 * vox) if density else B.Hierarchy(vox, 4, "elastic")
    H.solve(_load(H), precision="f64" if density else "f32", tol=1e-3)
    sizes = {_stencil_bytes(H, l) for l in (2, 3)} | {2 * _stencil_bytes(H, l) - 16 for l in (2, 3)}
    assert not sizes & set(H._arena.made)
    H.close()
