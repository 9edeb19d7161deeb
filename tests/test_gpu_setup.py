"""GPU parity of the hierarchy build's kernels at the sizes where they can go wrong: the inverse of
the pinned coarsest operator (tile and panel remainders, the smallest and largest matrices), the
staged sweep's tables (periodic wraps, both routes), the component count (runs across the period)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gmt_inputs import gyroid_sheet, laminate, uniform  # noqa: E402
from oracle import hierarchy as ohier  # noqa: E402
from oracle import solve as osolve  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _gmt():
    from paper_2604_26518_amd import binding
    return binding


# rows: 8 (padded to one 32-row tile), 81, 375 and 1029 (remainders of tile and panel), 1536 (none),
# 1728, and 2048 - the largest accepted; levels 1 (shared K_e), 2 (mask table) and 3 (per element)
COARSE = {
    "thermal2": (lambda: uniform(2), 1, "thermal"),
    "elastic3": (lambda: uniform(3), 1, "elastic"),
    "elastic5": (lambda: uniform(5), 1, "elastic"),
    "elastic8": (lambda: uniform(8), 1, "elastic"),
    "thermal12": (lambda: uniform(12), 1, "thermal"),
    "gyroid14": (lambda: gyroid_sheet(14, 1, 0.5), 2, "elastic"),
    "gyroid28": (lambda: gyroid_sheet(28, 4, 0.35), 3, "elastic"),
    "gyroid40_th": (lambda: gyroid_sheet(40, 2, 0.3), 3, "thermal"),
}


@pytest.mark.parametrize("case", sorted(COARSE))
def test_coarsest_inverse(case):
    """coarse_solve against a direct solve of the oracle's matrix.  Either side's solution is within
    n eps cond(K) of exact (Cholesky factor and its inverse), hence the bound."""
    make, L, phys = COARSE[case]
    vox = make()
    P = osolve.Problem(vox, L, phys)
    H = _gmt().Hierarchy(vox, L, phys)
    n = P.levels[-1].n_n
    f = np.random.default_rng(7).standard_normal((n, H.c, H.d))
    u = H.coarse_solve(torch.as_tensor(f, device=DEV)).cpu().numpy()
    ref = osolve.coarse_solve(P, f)
    assert np.all(u[0] == 0)
    A = _pinned(H, L)
    w = np.linalg.eigvalsh(A)
    bound = 4 * A.shape[0] * np.finfo(float).eps * w[-1] / w[0]
    err = np.linalg.norm(u - ref) / np.linalg.norm(ref)
    print(f"[{case}] rows {n * H.d} error {err:.1e} bound {bound:.1e}", flush=True)
    assert err <= bound
    # the inverse is symmetric bit for bit: x . (inv y) for unit vectors
    if n * H.d <= 400:
        inv = np.stack([_column(H, j) for j in range(n * H.d)], 1)
        assert np.array_equal(inv, inv.T)


def _pinned(H, L):
    m = H.export_maps(L)
    K = H.export_element_matrices(L).cpu().numpy()
    en = m["elem_nodes"].cpu().numpy()
    D, n = H.d, H.n_n(L)
    dof = (en[:, :, None] * D + np.arange(D)).reshape(en.shape[0], -1)
    A = np.zeros((n * D, n * D))
    np.add.at(A, (dof[:, :, None], dof[:, None, :]), K)
    return A[D:, D:]


def _column(H, j):
    n = H.n_n(H.L)
    f = np.zeros((n, H.c, H.d))
    f[j // H.d, 0, j % H.d] = 1.0
    return H.coarse_solve(torch.as_tensor(f, device=DEV)).cpu().numpy()[:, 0, :].reshape(-1)


def test_coarsest_size_limit():
    """2048 rows are accepted, more are refused before any work on them."""
    B = _gmt()
    vox = np.zeros((13, 13, 13), dtype=np.uint8)
    vox[:, :, :12] = 1  # 13^3 = 2197 nodes
    with pytest.raises(B.GmtError) as ei:
        B.Hierarchy(vox, 1, "thermal")
    assert ei.value.status == B.GMT_E_INVAL and "2197 DOFs" in str(ei.value)


@pytest.mark.parametrize("nodes", [256, 512])
@pytest.mark.parametrize("case", ["uniform4", "uniform18", "gyroid32", "laminate20"])
def test_stage_tables_routes(case, nodes, monkeypatch):
    """The staged sweep's tables from the bitmap and from the sorted groups are the same: the residual
    is bit for bit the same, with every group on one route, on the other, and with the bitmap too small
    for some groups only; and it is the plain interior sweep's (same products, same order)."""
    vox = {"uniform4": uniform(4), "uniform18": uniform(18), "gyroid32": gyroid_sheet(32, 0, 0.5),
           "laminate20": laminate(20, 7, axis=0)}[case]
    monkeypatch.setenv("GMT_STAGE_NODES", str(nodes))
    got = []
    for words in ("4096", "0", "40"):
        monkeypatch.setenv("GMT_STAGE_WORDS", words)
        H = _gmt().Hierarchy(vox, 4 if case == "gyroid32" else 2, "thermal" if case == "uniform18" else "elastic")
        u = torch.as_tensor(np.random.default_rng(3).standard_normal((H.n_n(), H.c, H.d)), device=DEV)
        for dt in (torch.float64, torch.float32):
            monkeypatch.setenv("GMT_FORCE_L1_VARIANT", "9")
            got.append(H.residual(H.load_vector(dt), u.to(dt)))
            monkeypatch.setenv("GMT_FORCE_L1_VARIANT", "7")
            assert torch.equal(got[-1], H.residual(H.load_vector(dt), u.to(dt)))
    for k in (2, 3, 4, 5):
        assert torch.equal(got[k], got[k % 2])


@pytest.mark.parametrize("N,L,fill", [(2, 1, 0.4), (5, 1, 0.1), (9, 1, 0.06), (18, 2, 0.03), (18, 2, 0.3), (64, 4, 0.04)])
def test_component_count(N, L, fill):
    """Random cells, each also with whole x-rows of voxels (runs that close on themselves)."""
    B = _gmt()
    for seed in range(4):
        rng = np.random.default_rng(seed)
        vox = (rng.random((N, N, N)) < fill).astype(np.uint8)
        if seed % 2:
            vox[rng.integers(N), rng.integers(N), :] = 1
        vox[0, 0, 0] = 1
        want = ohier.node_components(vox)
        try:
            B.Hierarchy(vox, L, "thermal").close()
            message = ""
        except B.GmtError as e:
            message = str(e)
        assert (f"form {want} node-connected components" in message) == (want != 1), (N, fill, seed, want, message)
        assert want != 1 or "components" not in message


@pytest.mark.parametrize("rows", [2048, 2049])
def test_coarsest_at_the_limit(rows):
    """The largest matrix (64 full tiles) is inverted, one row more is refused."""
    B = _gmt()
    vox = np.zeros((16, 16, 16), dtype=np.uint8)
    nodes = set()
    for z, y, x in np.ndindex(12, 13, 13):  # voxel by voxel, each touching the ones before
        corners = {(z + c // 4, y + c // 2 % 2, x + c % 2) for c in range(8)}
        if len(nodes | corners) <= rows:
            nodes |= corners
            vox[z, y, x] = 1
    assert len(nodes) == rows
    if rows > 2048:
        with pytest.raises(B.GmtError, match=f"{rows} DOFs") as ei:
            B.Hierarchy(vox, 1, "thermal")
        assert ei.value.status == B.GMT_E_INVAL
        return
    H = B.Hierarchy(vox, 1, "thermal")
    assert H.n_n(1) == rows
    f = np.random.default_rng(7).standard_normal((rows, H.c, H.d))
    u = H.coarse_solve(torch.as_tensor(f, device=DEV)).cpu().numpy()
    A = _pinned(H, 1)
    w = np.linalg.eigvalsh(A)
    ref = np.linalg.solve(A, f[1:, :, 0])
    err = np.linalg.norm(u[1:, :, 0] - ref) / np.linalg.norm(ref)
    bound = 4 * A.shape[0] * np.finfo(float).eps * w[-1] / w[0]
    print(f"[rows {rows}] error {err:.1e} bound {bound:.1e}", flush=True)
    assert np.all(u[0] == 0) and err <= bound
    H.close()
