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


class Budget(Recorder):
    """No more than `limit` bytes live over all arenas (None: any number); `peak`: the most there were."""

    limit = None
    live_bytes = 0
    peak = 0

    def _alloc(self, nbytes, ctx):
        if Budget.limit is not None and Budget.live_bytes + int(nbytes) > Budget.limit:
            return None
        ptr = super()._alloc(nbytes, ctx)
        if ptr is not None:
            Budget.live_bytes += int(nbytes)
            Budget.peak = max(Budget.peak, Budget.live_bytes)
        return ptr

    def _release(self, ptr, ctx):
        Budget.live_bytes -= self.size.get(ptr, 0)
        super()._release(ptr, ctx)


@pytest.fixture
def budget(monkeypatch):
    monkeypatch.setattr(B, "_TorchArena", Budget)
    monkeypatch.setattr(Budget, "limit", None)
    monkeypatch.setattr(Budget, "live_bytes", 0)
    monkeypatch.setattr(Budget, "peak", 0)
    return Budget


def _run(batch, graph, limit=None):
    """Mixed solves that go on with the FP64 recurrence after two FP32 iterations.  Returns the residuals,
    whether every cell had stencils, and the most bytes that the solves had live."""
    hs = [B.Hierarchy(gyroid_sheet(32, s, 0.3), 4, "elastic") for s in ((0, 1, 2) if batch else (0,))]
    fs = [H.load_vector() for H in hs]
    Budget.peak, Budget.limit = Budget.live_bytes, limit
    if batch:
        us, reps = B.solve_batch(hs, fs, tol=1e-8, precision="f32", n_workers=2, graph=graph)
    else:
        us, reps = zip(*[H.solve(f, tol=1e-8, precision="f32", graph=graph) for H, f in zip(hs, fs)])
    peak, Budget.limit = Budget.peak, None
    stencils = [any(_stencil_bytes(H, l) in H._arena.made for l in (2, 3)) for H in hs]
    rel = [float(max(H.relative_residual(f, u))) for H, f, u in zip(hs, fs, us)]
    assert all(r["converged"] for r in reps)
    for H in hs:
        H.close()
    return max(rel), stencils, peak


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("batch", [False, True])
def test_stencils_make_room(batch, graph, budget, monkeypatch):
    """Solves succeed in the memory that they take without stencils: the buffers of the FP64 recurrence
    have the room of stencils laid out before.  The batch has no other memory than the callback's."""
    monkeypatch.setenv("GMT_MAX_INNER32", "2")
    if batch:
        monkeypatch.setenv("GMT_HIP_ALLOC_MAX", "4096")
    monkeypatch.setenv("GMT_FORCE_COARSE_VARIANT", "1")  # element matrices
    rel, stencils, peak = _run(batch, graph)
    assert rel <= 1e-8 and not any(stencils)
    monkeypatch.setenv("GMT_FORCE_COARSE_VARIANT", "4")  # stencils, as long as they are held
    rel, stencils, _ = _run(batch, graph, limit=peak)
    assert rel <= 1e-8 and all(stencils)


def test_time_sweep_times_the_solvers_sweep(monkeypatch):
    """On a coarse level that is the stencil sweep where solves take one: timing lays it out."""
    monkeypatch.setattr(B, "_TorchArena", Recorder)
    monkeypatch.setenv("GMT_FORCE_COARSE_VARIANT", "5")
    H = B.Hierarchy(gyroid_sheet(32, 0, 0.3), 4, "elastic")
    assert H.time_sweep(2, reps=3) > 0
    assert _stencil_bytes(H, 2) in H._arena.size.values()
    H.close()
