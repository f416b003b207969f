"""The flux pass's small tiles where a tile has more edges than slots: cells in
the order of their number of neighbours, so that the last tile owns few of its
many edges (its border overflows) or the first more than it has slots for.  The
same bytes as with the large tiles."""
import numpy as np
import pytest

import parity_util as U  # noqa: F401  (puts the package on the path)
from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import tess as T

pytestmark = pytest.mark.gpu

TILE = 64


@pytest.mark.parametrize("riemann", [0, 1])
@pytest.mark.parametrize("falling", [0, 1])
@pytest.mark.parametrize("name", ["sod", "wave"])
def test_more_edges_than_slots(name, falling, riemann):
    import torch
    from paper_1410_3219_amd import rich as R
    P = {"sod": I.sod, "wave": I.advected_wave}[name](k=16, seed=3)
    g = np.random.default_rng(7)
    x, y = (P.box[a] + (P.box[2 + a] - P.box[a]) * g.uniform(1e-3, 1 - 1e-3, 2000) for a in (0, 1))
    m = T.rich_tess_build(x, y, P.box, P.bc)
    o = np.argsort(np.diff(m.off), kind="stable")
    o = o[::-1] if falling else o
    m = T.rich_tess_build(np.ascontiguousarray(x[o]), np.ascontiguousarray(y[o]), P.box, P.bc)
    n = m.n_cells
    first = 0 if falling else (n - 1) // TILE * TILE - TILE   # (a full tile)
    edges = np.unique(np.asarray(m.idx[m.off[first]:m.off[first + TILE]]) >> 1)
    owned = m.eoff[first + TILE] - m.eoff[first]
    assert len(edges) > 448 and (owned > 200 if falling else len(edges) - owned > 384)
    rho = g.uniform(0.5, 1.0, n)
    v, p = g.uniform(-0.2, 0.2, (2, n)), rho * g.uniform(0.9, 1.1, n)
    M = rho * m.area
    Q = np.stack([M, M * v[0], M * v[1], m.area * p / (P.gamma - 1) + 0.5 * M * (v ** 2).sum(0)])
    dm, s = R.DeviceMesh.from_host(m), R.DeviceState.from_host(Q, np.stack([m.px, m.py]))
    small, large = R.DeviceState.empty_like(s), R.DeviceState.empty_like(s)
    par, ws, wb = R.Params(gamma=P.gamma, riemann=riemann), R.workspace(n), R.batch_workspace([n])
    R.rich_stage(dm, s, s, small, 1e-5, par, ws)
    assert R.rich_stage_flags(ws) == 0
    plan = R.rich_stage_batch_prepare_tile([dm], [s], [s], [large], [1e-5], [par], 256, wb)
    R.rich_stage_batch_launch(plan, wb)
    assert R.rich_batch_flags(1, wb) == [0]
    torch.cuda.synchronize()
    assert torch.equal(small.Q, large.Q) and torch.equal(small.X, large.X)
