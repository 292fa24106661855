"""The candidate records of a velocity field's pair sum: every launch shape at
sizes that fill no tile, after a build, after steps, after a state was loaded
and after an adjoint, where the records are made again from the arrays.

Against the FP64 oracle: 1e-12 (FP64) and 1e-5 (FP32) relative L2, as for the
right-hand side elsewhere.  A resumed run and one that an adjoint left are the
same, bit for bit, as the run that only stepped.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2108_09488_amd import _lib
from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("integrator", [_lib.ADE_EULER, _lib.ADE_PC])
@pytest.mark.parametrize("dim,rb,n_side", [(2, 4, 23), (2, 8, 17), (3, 4, 10), (3, 8, 9)])
def test_records_follow_the_state(dim, rb, n_side, integrator):
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg1" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=1.4, jitter=0.1,
                    dt=2.0 ** -12)
    x = spec.positions()
    real = np.float32 if rb == 4 else np.float64
    C = spec.concentration(x).astype(real)
    v = I.velocity_field(x, spec.L, quantum=2.0 ** -20).astype(real).astype(np.float64)
    ref = O.rhs(O.model_from_spec(spec), x, C.astype(np.float64), v=v, mass=spec.mass, rho=spec.rho0)
    p = params_from_spec(spec, integrator=integrator, flags=_lib.ADE_VELOCITY_FIELD)

    def fresh(lanes):
        c = Context([p], [spec.n])
        c.init(torch.from_numpy(x), torch.from_numpy(C)).set_velocities(torch.from_numpy(v)).build()
        c.set_tuning(block=64, lanes=lanes)
        return c

    for lanes in (1, 2, 4):
        print(f"[case] records dim={dim} rb={rb} integ={integrator} lanes={lanes}", flush=True)
        a = fresh(lanes)
        r = a.rhs().double().cpu().numpy()
        assert np.linalg.norm(r - ref) / np.linalg.norm(ref) < (1e-12 if rb == 8 else 1e-5)
        a.step(3)
        state = a.save_state()
        ra = a.rhs().cpu().numpy()
        a.step(2)
        Ca = a.read_C().cpu().numpy()
        b = Context([p], [spec.n])
        b.load_state(state)
        b.set_tuning(block=64, lanes=lanes)
        assert np.array_equal(b.rhs().cpu().numpy(), ra)
        b.step(2)
        assert np.array_equal(b.read_C().cpu().numpy(), Ca)
        d = fresh(lanes)
        xs = torch.from_numpy(np.ascontiguousarray(x[:, :5]))
        d.adjoint(3, 2, xs, torch.zeros(5, dtype=torch.float32 if rb == 4 else torch.float64))
        assert np.array_equal(d.rhs().cpu().numpy(), ra)
        d.step(2)
        assert np.array_equal(d.read_C().cpu().numpy(), Ca)
        assert d.info()["step"] == a.info()["step"] == 5
        for c in (a, b, d):
            c.close()


@pytest.mark.parametrize("integrator", [_lib.ADE_EULER, _lib.ADE_PC])
@pytest.mark.parametrize("dim,rb,n_side", [(2, 4, 21), (2, 8, 16), (3, 4, 10), (3, 8, 9)])
def test_field_adjoint_of_any_checkpoint_interval(dim, rb, n_side, integrator):
    """The states that the adjoint keeps and runs again depend on the checkpoint
    interval, what it computes does not: J, the gradient and the state it leaves
    are the same bits for every interval, and the state is that of the steps."""
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg1" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=1.4, jitter=0.1,
                    dt=2.0 ** -12)
    x = spec.positions()
    real = np.float32 if rb == 4 else np.float64
    C = spec.concentration(x).astype(real)
    v = I.velocity_field(x, spec.L, quantum=2.0 ** -20).astype(real).astype(np.float64)
    xs = torch.from_numpy(np.ascontiguousarray(x[:, :7]))
    obs = torch.full((7,), 0.25, dtype=torch.float32 if rb == 4 else torch.float64)
    ctx = Context([params_from_spec(spec, integrator=integrator, flags=_lib.ADE_VELOCITY_FIELD)], [spec.n])

    def start():
        ctx.init(torch.from_numpy(x), torch.from_numpy(C)).set_velocities(torch.from_numpy(v)).build()

    for nsteps in (1, 2, 5):
        start()
        ctx.step(nsteps)
        want = (ctx.read_C().cpu().numpy(), ctx.read_x().cpu().numpy(), ctx.rhs().cpu().numpy())
        first = None
        for K in (nsteps, 1, 2, 3, 9):
            print(f"[case] field adjoint dim={dim} rb={rb} integ={integrator} steps={nsteps} K={K}", flush=True)
            start()
            J, g = ctx.adjoint(nsteps, K, xs, obs)
            assert ctx.info()["step"] == nsteps
            for a, b in zip((ctx.read_C(), ctx.read_x(), ctx.rhs()), want):
                assert np.array_equal(a.cpu().numpy(), b), (nsteps, K)
            got = (J, *[float(t) for t in g])
            first = first or got
            assert got == first, (nsteps, K)
            assert np.isfinite(got).all() and any(t != 0.0 for t in got[1:])
    ctx.close()
