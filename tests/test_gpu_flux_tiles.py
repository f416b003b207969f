"""The flux pass's small tiles (64 cells and four threads per cell, taken by
launches of under 81 920 cells) against the large ones (256 cells): the same
bytes, at meshes of less than a tile, a tile, a tile and one cell, and several,
with both solvers and boundaries, and where most of a tile's edges belong to
others (cells in random order), which overflows its list of them."""
import numpy as np
import pytest

import parity_util as U  # noqa: F401  (puts the package on the path)
from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import tess as T

pytestmark = pytest.mark.gpu


def _mesh(name, nx, ny, shuffled):
    """nx * ny cells of a problem's box, jittered; in its order or shuffled."""
    P = (I.sod if name == "sod" else I.advected_wave)(k=16, seed=3)
    g = np.random.default_rng(7)
    x0, y0, x1, y1 = P.box
    gx, gy = np.meshgrid((np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny, indexing="ij")
    px = x0 + (x1 - x0) * (gx + g.uniform(-0.2, 0.2, gx.shape) / nx).ravel()
    py = y0 + (y1 - y0) * (gy + g.uniform(-0.2, 0.2, gy.shape) / ny).ravel()
    if shuffled:
        o = g.permutation(len(px))
    else:
        o = T.rich_tess_hilbert_order(px, py, P.box)
    m = T.rich_tess_build(px[o], py[o], P.box, P.bc)
    rho = np.where(m.px < 0.5 * (x0 + x1), 1.0, 0.3) * g.uniform(0.9, 1.1, m.n_cells)
    v, p = g.uniform(-0.2, 0.2, (2, m.n_cells)), rho * g.uniform(0.9, 1.1, m.n_cells)
    M = rho * m.area
    Q = np.stack([M, M * v[0], M * v[1], m.area * p / (P.gamma - 1) + 0.5 * M * (v ** 2).sum(0)])
    return P, m, Q, np.stack([m.px, m.py])


@pytest.mark.parametrize("riemann", [0, 1])
@pytest.mark.parametrize("name,nx,ny,shuffled", [("wave", 7, 9, 0), ("sod", 8, 8, 0),
                                                 ("sod", 5, 13, 0), ("wave", 31, 33, 0),
                                                 ("sod", 40, 40, 1), ("wave", 40, 41, 1)])
def test_small_and_large_tiles_agree_bitwise(name, nx, ny, shuffled, riemann):
    import torch
    from paper_1410_3219_amd import rich as R
    P, m, Q, X = _mesh(name, nx, ny, shuffled)
    dm = R.DeviceMesh.from_host(m)
    s = R.DeviceState.from_host(Q, X)
    p = R.Params(gamma=P.gamma, riemann=riemann)
    h = 0.05 / max(nx, ny)
    one, two, big = (R.DeviceState.empty_like(s) for _ in range(3))
    ws = R.workspace(m.n_cells)
    R.rich_stage(dm, s, s, one, h, p, ws)                      # 64-cell tiles
    assert R.rich_stage_flags(ws) == 0
    wb = R.batch_workspace([m.n_cells])
    R.rich_stage_batch([dm], [s], [s], [two], [h], [p], wb)    # the same in a batch
    assert R.rich_batch_flags(1, wb) == [0]
    plan = R.rich_stage_batch_prepare_tile([dm], [s], [s], [big], [h], [p], 256, wb)
    R.rich_stage_batch_launch(plan, wb)
    assert R.rich_batch_flags(1, wb) == [0]
    torch.cuda.synchronize()
    for o in (one, two):
        assert torch.equal(o.Q, big.Q) and torch.equal(o.X, big.X)


def test_plan_reports_and_takes_the_offered_shapes_only():
    """A small batch's default plan reports a shape that the explicit call takes
    back; the shapes that are not offered are refused by both explicit calls."""
    from paper_1410_3219_amd import rich as R
    P, m, Q, X = _mesh("sod", 8, 8, 0)
    dm, s = R.DeviceMesh.from_host(m), R.DeviceState.from_host(Q, X)
    out = R.DeviceState.empty_like(s)
    a = [dm], [s], [s], [out], [1e-3], [R.Params(gamma=P.gamma)]
    wb = R.batch_workspace([m.n_cells])
    tile = R.rich_stage_batch_prepare(*a, wb).flux_tile
    assert R.rich_stage_batch_prepare_tile(*a, tile, wb).flux_tile == tile
    for bad in (-1, 0, 64, 96):
        for call in (lambda: R.rich_stage_batch_prepare_tile(*a, bad, wb),
                     lambda: R.rich_stage_batch_prepare_courant(*a, wb, tile=bad)):
            with pytest.raises(R.RichError) as e:
                call()
            assert e.value.status == R.RICH_E_INVAL
