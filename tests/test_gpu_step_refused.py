"""Calls that the step drivers refuse: what a stage refuses, both of them do; and
runs whose meshes the device rebuild does not take (a periodic box of under 16
cells) or does not certify (a cell of more neighbours than it holds): their
meshes come from the host stage, and the other runs of a batch are as if alone."""
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


def _steps_equal(R, cases, dts, n_steps, integrator=0):
    """Steps of the cases as one batch and each alone: the same bits; the
    counts of device-built and host-built meshes of the batch and alone."""
    batch, alone = ([_run(R, c) for c in cases] for _ in range(2))
    ps = [R.Params(gamma=c[0].gamma, integrator=integrator) for c in cases]
    ws = R.batch_workspace([c[1].n_cells for c in cases])
    for _ in range(n_steps):
        st = R.rich_step_batch([b[0] for b in batch], [b[1] for b in batch], dts, ps, ws)
        assert st == [R.RICH_OK] * len(cases)
        for a, dt, p in zip(alone, dts, ps):
            a[0].step(a[1], dt, p)
    for a, b in zip(alone, batch):
        for u, v in zip(a[1].numpy(), b[1].numpy()):
            assert np.array_equal(u, v)
    return [b[0].tess_counts() for b in batch], [a[0].tess_counts() for a in alone]


@pytest.mark.parametrize("integrator", [0, 1])
def test_a_run_the_rebuild_does_not_take_leaves_the_others_alone(integrator):
    from paper_1410_3219_amd import rich as R
    cases = [_problem("sod", 20), _problem("wave", 3), _problem("gresho", 24)]
    batch, alone = _steps_equal(R, cases, [1e-3] * 3, 2, integrator)
    k = 2 * (2 - integrator)
    assert batch == alone == [(k, 0), (0, k), (k, 0)]


def _hub(petals=20):
    """A point at rest inside a ring of 20: more neighbours than the device
    rebuild holds, before and after every step."""
    P = I.sod(k=20, seed=4)
    keep = np.hypot(P.px - 0.5, P.py - 0.5) > 0.1
    a = 2 * np.pi * np.arange(petals) / petals
    m = T.rich_tess_build(np.concatenate([P.px[keep], [0.5], 0.5 + 0.06 * np.cos(a)]),
                          np.concatenate([P.py[keep], [0.5], 0.5 + 0.06 * np.sin(a)]), P.box, P.bc)
    assert np.diff(m.off).max() == petals
    return P, m, I.conserved(1.0, 0.0, 0.0, 1.0, m.area, P.gamma)


def test_a_run_whose_rebuild_fails_leaves_the_others_alone():
    from paper_1410_3219_amd import rich as R
    cases = [_problem("sod", 20), _hub(), _problem("gresho", 24)]
    batch, alone = _steps_equal(R, cases, [1e-3, 1e-5, 1e-3], 3)
    assert batch == alone == [(6, 0), (0, 6), (6, 0)]
