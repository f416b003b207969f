"""The two ways the device re-tessellation proves a cell whose neighbours
stayed: in one launch (small calls), or the ring first and the neighbours'
neighbours only of cells with a failed neighbour (calls of 98 304 cells and
more).  A run rebuilt alone takes the first, the same run beside a filler of
102 400 cells the second; both must give the same bytes (or refuse with the same
counts), whatever the mesh and however far its points moved."""
import math

import numpy as np
import pytest

from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import tess as T

pytestmark = pytest.mark.gpu

MAKE = {"wave": I.advected_wave, "sod": I.sod, "sedov": I.sedov, "gresho": I.gresho}


def _mesh(name, k):
    """A problem's mesh, or one of uniformly random points in its box."""
    if name in MAKE:
        P = MAKE[name](k=k, seed=2)
        return T.rich_tess_build(P.px, P.py, P.box, P.bc)
    P = (I.advected_wave if name == "random_periodic" else I.sod)(k=k, seed=2)
    g = np.random.default_rng(11)
    x, y = (P.box[a] + (P.box[2 + a] - P.box[a]) * g.uniform(1e-4, 1 - 1e-4, k * k)
            for a in (0, 1))
    return T.rich_tess_build(x, y, P.box, P.bc)


def _moved(m, move):
    h = math.sqrt((m.box[2] - m.box[0]) * (m.box[3] - m.box[1]) / m.n_cells)
    X = np.stack([m.px, m.py]) + h * np.random.default_rng(5).uniform(-move, move, (2, m.n_cells))
    for a in (0, 1):
        lo, hi = m.box[a], m.box[2 + a]
        X[a] = lo + np.mod(X[a] - lo, hi - lo) if m.bc == T.BC_PERIODIC else \
            np.clip(X[a], lo + 1e-3 * h, hi - 1e-3 * h)
    return X


def _bytes(b, info):
    t = {k: v.cpu().numpy() for k, v in b.t.items()}
    return [t["cells"].tobytes(), t["off"].tobytes(), t["eoff"].tobytes(),
            t["idx"][:info["n_csr"]].tobytes(), t["edges"][:32 * info["n_edges"]].tobytes()]


@pytest.mark.parametrize("move", [0.0, 0.02, 0.1])
@pytest.mark.parametrize("name,k", [("wave", 8), ("wave", 61), ("sod", 9), ("sod", 63),
                                    ("sedov", 40), ("gresho", 50), ("random_periodic", 47),
                                    ("random_walls", 47)])
def test_both_paths_give_the_same_mesh(name, k, move):
    import torch
    from paper_1410_3219_amd import rich as R
    hosts = [_mesh(name, k), _mesh("wave", 320)]
    Xs = [torch.from_numpy(_moved(m, move)).cuda() for m in hosts]
    prevs = [R.DeviceMesh.from_host(m) for m in hosts]

    def buffers():
        return ([R.DeviceMeshBufs(m.n_cells, m.box, m.bc) for m in hosts],
                [R.retess_workspace(m.n_cells) for m in hosts])

    alone, ws = buffers()
    R.rich_retess(prevs[0], Xs[0], alone[0], ws[0])
    st, info = R.rich_retess_result(ws[0])
    # (random points moved far gain neighbours that are no candidates: refused)
    assert st == R.RICH_OK or (name.startswith("random") and move > 0), info
    both, ws = buffers()
    bws = R.rich_retess_batch(prevs, Xs, both, ws)
    res = R.rich_retess_batch_result(2, bws)
    assert res[0] == (st, info) and res[1][0] == R.RICH_OK, res
    if st == R.RICH_OK:
        assert _bytes(both[0], info) == _bytes(alone[0], info)
    # alone and large: the second path's launches of a single run
    R.rich_retess(prevs[1], Xs[1], alone[1], ws[1])
    st1, info1 = R.rich_retess_result(ws[1])
    assert (st1, info1) == res[1]
    assert _bytes(alone[1], info1) == _bytes(both[1], info1)


@pytest.mark.parametrize("name,k", [("wave", 40), ("sod", 41), ("random_walls", 40)])
def test_stored_and_recomputed_geometry_agree(name, k):
    """In a box whose coordinates are large against its cells the cells' edges
    are stored and compared; elsewhere they are recomputed from the points.
    The same points (on a grid of 2^-30, so that the shift by 2048 is exact)
    give the same indices either way, and lengths and midpoints to rounding:
    1e-13 of a unit box for values computed alike up to the order of a few
    operations, plus the 2.3e-13 that a coordinate near 2048 is rounded by."""
    import torch
    from paper_1410_3219_amd import rich as R
    grid = 2.0 ** -30
    m = _mesh(name, k)
    pts = np.round(np.stack([m.px, m.py]) / grid) * grid
    new = np.round(_moved(m, 0.0 if name.startswith("random") else 0.02) / grid) * grid
    out = []
    for s in (0.0, 2048.0):
        h = T.rich_tess_build(pts[0] + s, pts[1] + s, [v + s for v in m.box], m.bc)
        X = torch.from_numpy(new + s).cuda()
        b, ws = R.DeviceMeshBufs(h.n_cells, h.box, h.bc), R.retess_workspace(h.n_cells)
        R.rich_retess(R.DeviceMesh.from_host(h), X, b, ws)
        st, info = R.rich_retess_result(ws)
        assert st == R.RICH_OK, info
        t = {q: v.cpu().numpy() for q, v in b.t.items()}
        e = t["edges"][:32 * info["n_edges"]].view(np.float64).reshape(-1, 4)
        out.append((t["off"], t["eoff"], t["idx"][:info["n_csr"]],
                    e.view(np.int32).reshape(-1, 8)[:, 6:], e[:, :2] - s, e[:, 2]))
    for a, b in zip(out[0][:4], out[1][:4]):
        assert np.array_equal(a, b)
    assert np.abs(out[0][5] - out[1][5]).max() < 1e-13
    assert np.abs(out[0][4] - out[1][4]).max() < 1e-13 + 2.3e-13
