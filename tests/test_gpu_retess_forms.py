"""Which of the device re-tessellation's two forms a run takes (one launch that
tries every candidate, or the ring first and the neighbours' neighbours only of
cells with a failed neighbour) follows from the run alone: its companions in a
batch, and how much room its previous mesh's buffers have, change no bit.

The forms differ in one place: a neighbour's neighbour that is inside a vertex's
circle by the margin of the cell's own test (1e-9 of the candidate's half squared
distance plus the largest squared vertex distance) but outside it by those of
the neighbours' tests.  The first form sends that cell to the clip, the second
does not; the meshes here have such a point."""
import math

import numpy as np
import pytest

from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import tess as T
import test_gpu_retess as G

pytestmark = pytest.mark.gpu

MASK = 0x0FFFFFFF
MARGIN = 1e-9


def _ring(m, c):
    """Neighbours of cell c, counter-clockwise; None where not all are plain."""
    ent = np.asarray(m.idx[m.off[c]:m.off[c + 1]], dtype=np.int64)
    u = np.asarray(m.e_j, dtype=np.int64)[ent >> 1] & 0xFFFFFFFF
    if (u >> 28).any():
        return None
    return [int(v) for v in np.where(ent & 1, np.asarray(m.e_i)[ent >> 1], u & MASK)]


def _centre(p, a, b, c):
    """Circumcentre of points a, b, c relative to point a."""
    u, v = p[b] - p[a], p[c] - p[a]
    return np.array([v[1] * (u @ u) - u[1] * (v @ v), u[0] * (v @ v) - v[0] * (u @ u)]) / (
        2 * (u[0] * v[1] - u[1] * v[0]))


def _window(m, p, i, a, b, k):
    """How far k is outside the circle of i, a, b (half its power), and the
    margins between which it has to lie: above those of the tests at a and b,
    below that of the test at i.  (i seen from k's circle: scaled alike.)"""
    def reach2(c):
        r = _ring(m, c)
        return max(np.sum(_centre(p, c, u, v) ** 2) for u, v in zip(r, r[1:] + r[:1]))

    def slack(o, s, t, w):   # w against the circle of o, s, t
        u = p[w] - p[o]
        return 0.5 * (u @ u) - _centre(p, o, s, t) @ u

    def margin(o, w):
        return MARGIN * (0.5 * np.sum((p[w] - p[o]) ** 2) + reach2(o))

    s, back = slack(i, a, b, k), slack(k, a, b, i)
    low = max(max(margin(c, k), margin(c, i) * s / back) for c in (a, b))
    return s, low, margin(i, k)


def _planted(name, k, seed=2):
    """A problem's mesh of k x k points, one moved so that it lies between the
    margins at some cell."""
    P = {"wave": I.advected_wave, "sod": I.sod}[name](k=k, seed=seed)
    m = T.rich_tess_build(P.px, P.py, P.box, P.bc)
    p = np.stack([m.px, m.py], axis=1)
    lo, hi = 0.4, 0.6
    inside = np.flatnonzero(((p > lo) & (p < hi)).all(axis=1))[:400]
    found = []
    for a in inside:
        r = _ring(m, a)
        for q, b in enumerate(r):
            i, w = r[q - 1], r[(q + 1) % len(r)]
            if a < b and ((p[[i, b, w]] > lo) & (p[[i, b, w]] < hi)).all():
                u = p[w] - p[i]
                s = 0.5 * (u @ u) - _centre(p, i, a, b) @ u
                found.append((s / (u @ u), i, a, b, w))
    for _, i, a, b, w in sorted(found)[:40]:
        if any(_ring(m, c) is None for c in (i, a, b, w)):
            continue
        s, low, high = _window(m, p, i, a, b, w)
        if not low > 0 or not high > 1.2 * low:
            continue
        q = p.copy()
        c = p[i] + _centre(p, i, a, b)
        d = p[w] - c
        r2 = np.sum((p[i] - c) ** 2)
        q[w] = c + d * math.sqrt((r2 + 2 * math.sqrt(low * high)) / (d @ d))
        n = T.rich_tess_build(q[:, 0].copy(), q[:, 1].copy(), P.box, P.bc)
        if not np.array_equal(n.px, q[:, 0]) or w not in (_ring(n, a) or []):
            continue
        s, low, high = _window(n, q, i, a, b, w)
        if 1.05 * low < s < high / 1.05:
            return n
    raise AssertionError("no such point")


def _points(m, move=0.0):
    import torch
    h = math.sqrt((m.box[2] - m.box[0]) * (m.box[3] - m.box[1]) / m.n_cells)
    X = np.stack([m.px, m.py]) + h * np.random.default_rng(5).uniform(-move, move, (2, m.n_cells))
    for a in (0, 1):
        lo, hi = m.box[a], m.box[2 + a]
        X[a] = lo + np.mod(X[a] - lo, hi - lo) if m.bc == T.BC_PERIODIC else \
            np.clip(X[a], lo + 1e-3 * h, hi - 1e-3 * h)
    return X, torch.from_numpy(X).cuda()


def _bytes(b, info):
    t = {k: v.cpu().numpy() for k, v in b.t.items()}
    return [t["cells"].tobytes(), t["off"].tobytes(), t["eoff"].tobytes(),
            t["idx"][:info["n_csr"]].tobytes(), t["edges"][:32 * info["n_edges"]].tobytes()]


def _rebuild(R, m, prev, X):
    b, ws = R.DeviceMeshBufs(m.n_cells, m.box, m.bc), R.retess_workspace(m.n_cells)
    R.rich_retess(prev, X, b, ws)
    st, info = R.rich_retess_result(ws)
    return st, info, b


@pytest.mark.parametrize("name", ["sod", "wave"])
def test_companions_change_no_bit(name):
    from paper_1410_3219_amd import rich as R
    hosts = [_planted(name, 61), _planted("wave", 320), _planted("sod", 60)]
    Xs = [_points(m)[1] for m in hosts]
    prevs = [R.DeviceMesh.from_host(m) for m in hosts]
    alone = [_rebuild(R, m, p, X) for m, p, X in zip(hosts, prevs, Xs)]
    assert all(a[0] == R.RICH_OK for a in alone), [a[1] for a in alone]
    assert alone[0][1]["n_clipped"] >= 1   # (the form of small runs: the point is inside its margin)
    bufs = [R.DeviceMeshBufs(m.n_cells, m.box, m.bc) for m in hosts]
    bws = R.rich_retess_batch(prevs, Xs, bufs, [R.retess_workspace(m.n_cells) for m in hosts])
    for (st, info), b, a in zip(R.rich_retess_batch_result(3, bws), bufs, alone):
        assert (st, info) == a[:2]
        assert _bytes(b, info) == _bytes(a[2], info)


@pytest.mark.parametrize("name", ["sod", "wave"])
def test_room_in_the_previous_buffers_changes_no_bit(name):
    import torch
    from paper_1410_3219_amd import rich as R
    m = _planted(name, 320)
    X = _points(m)[1]
    prev = R.DeviceMesh.from_host(m)
    st, info, b = _rebuild(R, m, prev, X)
    assert st == R.RICH_OK, info
    room = R.rich_retess_capacity(m.n_cells)[1] + 100000
    roomy = R.DeviceMesh(dict(prev.t), m.n_cells, m.n_edges, room, prev.box, prev.bc)
    roomy.t["idx"] = torch.zeros(room, dtype=torch.int32, device="cuda")
    roomy.t["idx"][:m.n_csr] = prev.t["idx"]
    st2, info2, b2 = _rebuild(R, m, roomy, X)
    assert (st2, info2) == (st, info)
    assert _bytes(b2, info2) == _bytes(b, info)


@pytest.mark.parametrize("move", [0.02, 0.1])
@pytest.mark.parametrize("name", ["sod", "wave"])
def test_large_single_runs_match_the_host_stage(name, move):
    """Single runs of 102 400 cells, between walls and periodic: every cell,
    edge and CSR entry of the input stage's mesh of the same points (1e-12 of
    the cell size, as the mesh of the benchmark's size)."""
    from paper_1410_3219_amd import rich as R
    P = {"wave": I.advected_wave, "sod": I.sod}[name](k=320, seed=3)
    m = T.rich_tess_build(P.px, P.py, P.box, P.bc)
    Xh, X = _points(m, move)
    st, info, b = _rebuild(R, m, R.DeviceMesh.from_host(m), X)
    assert st == R.RICH_OK and info["n_clipped"] > 0, info
    dev = R.mesh_to_host(b.mesh(), info["n_edges"], info["n_csr"])
    G.check_structure(dev)
    G.compare_meshes(dev, T.rich_tess_build(Xh[0], Xh[1], P.box, P.bc), 1.0 / 320)


def test_previous_mesh_of_more_entries_than_a_rebuilt_one():
    """A previous mesh that names neighbours twice, with more entries in use
    than a rebuilt mesh of its cells may have: taken as before, and the mesh is
    the same."""
    import torch
    from paper_1410_3219_amd import rich as R
    P = I.sod(k=320, seed=4)
    m = T.rich_tess_build(P.px, P.py, P.box, P.bc)
    off, idx = np.asarray(m.off, dtype=np.int64), np.asarray(m.idx)
    extra = R.rich_retess_capacity(m.n_cells)[1] + 1000 - m.n_csr
    deg = np.diff(off)
    more = np.zeros(m.n_cells, dtype=np.int64)
    wide = np.flatnonzero(deg <= 7)
    more[wide] = deg[wide]   # (every entry of these cells a second time)
    more[np.cumsum(more) > extra + 8] = 0
    assert more.sum() > extra and (deg + more).max() <= 14
    rows = [np.concatenate([idx[off[i]:off[i + 1]], idx[off[i]:off[i + 1]][:more[i]]])
            for i in range(m.n_cells)]
    prev = R.DeviceMesh.from_host(m)
    st, info, b = _rebuild(R, m, prev, _points(m, 0.02)[1])
    assert st == R.RICH_OK, info
    t = dict(prev.t)
    t["idx"] = torch.from_numpy(np.concatenate(rows).astype(np.int32)).cuda()
    t["off"] = torch.from_numpy(np.concatenate([[0], np.cumsum(deg + more)]).astype(np.int32)).cuda()
    twice = R.DeviceMesh(t, m.n_cells, m.n_edges, t["idx"].numel(), prev.box, prev.bc)
    st2, info2, b2 = _rebuild(R, m, twice, _points(m, 0.02)[1])
    assert st2 == R.RICH_OK, info2
    G.compare_meshes(R.mesh_to_host(b2.mesh(), info2["n_edges"], info2["n_csr"]),
                     R.mesh_to_host(b.mesh(), info["n_edges"], info["n_csr"]), 1.0 / 320)


def test_a_run_of_many_end_blocks_in_a_batch():
    """270 400 cells: more blocks of cells (265) than count on one word."""
    from paper_1410_3219_amd import rich as R
    hosts = []
    for name, k in (("wave", 520), ("sod", 20)):
        P = {"wave": I.advected_wave, "sod": I.sod}[name](k=k, seed=3)
        hosts.append(T.rich_tess_build(P.px, P.py, P.box, P.bc))
    Xs = [_points(m, 0.05)[1] for m in hosts]
    prevs = [R.DeviceMesh.from_host(m) for m in hosts]
    bufs = [R.DeviceMeshBufs(m.n_cells, m.box, m.bc) for m in hosts]
    bws = R.rich_retess_batch(prevs, Xs, bufs, [R.retess_workspace(m.n_cells) for m in hosts])
    for (st, info), b, m, p, X in zip(R.rich_retess_batch_result(2, bws), bufs, hosts, prevs, Xs):
        assert st == R.RICH_OK, info
        alone = _rebuild(R, m, p, X)
        assert (st, info) == alone[:2]
        assert _bytes(b, info) == _bytes(alone[2], info)


@pytest.mark.parametrize("noise", [1e-8, 0.02])
@pytest.mark.parametrize("name", ["sod", "wave"])
def test_large_exact_lattice_moves(name, noise):
    """An exact lattice of 102 400 cells whose points move by a part of the
    spacing: four cells met at each vertex of the previous mesh, so every cell
    gains neighbours that no ring holds.  The mesh is the input stage's (1e-12
    of the cell size), but for edges as short as the cut for dropping them."""
    import torch
    from paper_1410_3219_amd import rich as R
    P = {"wave": I.advected_wave, "sod": I.sod}[name](k=16, seed=3)
    k = 320
    c = (np.arange(k) + 0.5) / k
    x, y = (v.ravel() for v in np.meshgrid(c, c, indexing="ij"))   # (a unit box)
    assert tuple(P.box) == (0.0, 0.0, 1.0, 1.0)
    o = T.rich_tess_hilbert_order(x, y, P.box)
    m = T.rich_tess_build(x[o], y[o], P.box, P.bc)
    X = np.stack([m.px, m.py]) + noise / k * np.random.default_rng(5).uniform(-1, 1, (2, k * k))
    st, info, b = _rebuild(R, m, R.DeviceMesh.from_host(m), torch.from_numpy(X).cuda())
    assert st == R.RICH_OK, info
    dev = R.mesh_to_host(b.mesh(), info["n_edges"], info["n_csr"])
    G.check_structure(dev)
    ref = T.rich_tess_build(X[0], X[1], P.box, P.bc)
    (kd, *gd), (kr, *gr) = G.edge_keys(dev), G.edge_keys(ref)
    cut = 1e-12 / k / math.sqrt(math.pi)   # (edges of this length are kept or dropped by rounding)
    assert np.isin(kd[gd[0] > 2 * cut], kr).all() and np.isin(kr[gr[0] > 2 * cut], kd).all()
    both = np.intersect1d(kd, kr)
    assert len(both) > 2.9 * k * k
    for u, v in zip(gd, gr):   # lengths, midpoints
        assert np.abs(u[np.isin(kd, both)] - v[np.isin(kr, both)]).max() <= 1e-12 / k
    assert np.abs(dev.area - ref.area).max() <= 1e-12 / (k * k)
