"""Steps whose stages and mesh rebuilds are enqueued at once and read at their
end: a run that fails on the way (a step so long that a state turns
unphysical) returns what it returned before, with its state and mesh as they
were, beside runs that are committed and equal the same step taken alone; and
the Courant steps of many runs in one call."""
import numpy as np
import pytest

import parity_util as U  # noqa: F401  (puts the package on the path)
from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import tess as T

pytestmark = pytest.mark.gpu


def _run(R, name, k):
    P = {"sod": I.sod, "wave": I.advected_wave, "gresho": I.gresho}[name](k=k, seed=5)
    m = T.rich_tess_build(P.px, P.py, P.box, P.bc)
    ctx = R.RichCtx(device_tess=True)
    ctx.set_mesh(m)
    return ctx, R.DeviceState.from_host(P.state(m.area), np.stack([m.px, m.py])), P, m


@pytest.mark.parametrize("integrator,motion", [(0, 1), (0, 0), (1, 1)])
def test_failing_run_beside_good_ones(integrator, motion):
    import torch
    from paper_1410_3219_amd import rich as R
    names = [("sod", 20), ("wave", 17), ("gresho", 24)]
    batch = [_run(R, *x) for x in names]
    alone = [_run(R, *x) for x in names]
    ps = [R.Params(gamma=b[2].gamma, motion=motion, integrator=integrator) for b in batch]
    dts = [R.rich_cfl_dt(b[0].mesh(), b[1], p, R.workspace(b[3].n_cells))
           for b, p in zip(batch, ps)]
    dts[1] *= 1e4   # the wave's step
    before = batch[1][1].numpy()
    ws = R.batch_workspace([b[3].n_cells for b in batch])
    st = R.rich_step_batch([b[0] for b in batch], [b[1] for b in batch], dts, ps, ws)
    assert st[0] == st[2] == R.RICH_OK and st[1] == R.RICH_E_DOMAIN, st
    with pytest.raises(R.RichError) as err:
        alone[1][0].step(alone[1][1], dts[1], ps[1])
    assert err.value.status == R.RICH_E_DOMAIN
    for s in (batch[1][1], alone[1][1]):
        after = s.numpy()
        assert all(np.array_equal(a, b) for a, b in zip(before, after))
    for r in (0, 2):
        alone[r][0].step(alone[r][1], dts[r], ps[r])
        torch.cuda.synchronize()
        assert torch.equal(alone[r][1].Q, batch[r][1].Q)
        assert torch.equal(alone[r][1].X, batch[r][1].X)
        assert alone[r][0].tess_counts() == batch[r][0].tess_counts() == \
            ((2 - integrator) * motion, 0)
    # the failed run goes on from where it was
    dts[1] *= 1e-4
    assert R.rich_step_batch([batch[1][0]], [batch[1][1]], [dts[1]], [ps[1]], ws) == [R.RICH_OK]
    alone[1][0].step(alone[1][1], dts[1], ps[1])
    torch.cuda.synchronize()
    assert torch.equal(alone[1][1].Q, batch[1][1].Q)


def test_courant_steps_of_many_runs_equal_those_of_each():
    from paper_1410_3219_amd import rich as R
    runs = [_run(R, *x) for x in [("sod", 3), ("wave", 16), ("gresho", 33), ("sod", 90)]]
    ps = [R.Params(gamma=b[2].gamma, cfl=0.1 * (r + 1)) for r, b in enumerate(runs)]
    ws = R.batch_workspace([b[3].n_cells for b in runs])
    got = R.rich_cfl_dt_batch([b[0].mesh() for b in runs], [b[1] for b in runs], ps, ws)
    assert got == [R.rich_cfl_dt(b[0].mesh(), b[1], p, R.workspace(b[3].n_cells))
                   for b, p in zip(runs, ps)]
