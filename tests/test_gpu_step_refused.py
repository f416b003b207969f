"""Calls that the step drivers refuse: what a stage refuses, both of them do."""
import copy

import numpy as np
import pytest

import parity_util as U  # noqa: F401  (puts the package on the path)
from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import tess as T

pytestmark = pytest.mark.gpu


def _problem(name, k):
    P = {"sod": I.sod, "wave": I.advected_wave, "gresho": I.gresho}[name](k=k, seed=5)
    m = T.rich_tess_build(P.px, P.py, P.box, P.bc)
    return P, m, P.state(m.area)


def _run(R, case):
    P, m, Q = case
    ctx = R.RichCtx(device_tess=True)
    ctx.set_mesh(m)
    return ctx, R.DeviceState.from_host(Q, np.stack([m.px, m.py]))


@pytest.mark.parametrize("fault", ["box", "bc"])
def test_both_drivers_refuse_what_a_stage_refuses(fault):
    """A static mesh in an inverted box, or with a boundary kind there is not:
    refused by both drivers before anything is launched, the state untouched."""
    from paper_1410_3219_amd import rich as R
    P, m, Q = _problem("sod", 12)
    bad = copy.copy(m)
    if fault == "box":
        bad.box = (m.box[2], m.box[1], m.box[0], m.box[3])
    else:
        bad.bc = 7
    ctx, s = _run(R, (P, bad, Q))
    p = R.Params(gamma=P.gamma, motion=0)
    with pytest.raises(R.RichError) as e:
        ctx.step(s, 1e-4, p)
    assert e.value.status == R.RICH_E_INVAL
    ws = R.batch_workspace([m.n_cells])
    assert R.rich_step_batch([ctx], [s], [1e-4], [p], ws) == [R.RICH_E_INVAL]
    assert np.array_equal(s.numpy()[0], Q)
    assert np.array_equal(s.numpy()[1], np.stack([m.px, m.py]))
